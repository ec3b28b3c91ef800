// The Hadamard rotation in front of a quantized linear layer with the channel reorder absorbed into it (paper
// App. D, x H P), emitting y_P[m, j] = (x[m, :] H)[pi(j)] as a bf16 tensor, as the activation operand of the GEMM, or both.
//
// H = S_{2^k} (x) P_m / sqrt(K): channel i = a m + b (a: Sylvester index, natural order; b: Paley index).
// One wave, or the four of a workgroup, own a row.  The transform stays in registers:
//   1. m = 12, 20: the Paley factor is a matrix product of the bf16 row with the +-1 matrix, padded to the
//      tile of an MFMA instruction, straight from memory; its result lies with a in registers, lanes and
//      the wave's number.  m = 1: a lane loads 8 consecutive channels.
//   2. The Sylvester factor is sums and differences of values whose a differs in one bit, from the lowest
//      bit up: pairs of registers, or lanes of a wave by DPP exchanges (inside rows of 16) and swaps of
//      rows and halves.  A row of four waves meets once in LDS, for the last two bits.
//   3. Scaled, rounded to bf16 and put into the row's slab of LDS, from where the reordered row is gathered:
//      the reorder is the order in which the transform's output is consumed.
// The widths whose values do not fit a wave's registers that way (64 a lane) or leave it too few (below 8; 16 for
// m = 20) take the general path: passes over an fp32 row in LDS.
// Measured against one pass over LDS for each digit of 16 (of which the lowest met in few banks), us, NVFP4: 512 x 3072 6.2 ->
// 5.1, 4608 x 3072 22.4 -> 18.5, 4608 x 2048 29.3 -> 12.6, 8192 x 4096 104 -> 34, 4608 x 5120 43 -> 27, 2048 x 12288 41 -> 36.
// What bounds it: with few rows the chain; with many, besides the traffic (4608 x 3072: 36 MB), the vector unit -- sums,
// exchanges and the quantizer -- at four or five waves a SIMD; m = 12 and 20 leave a quarter and three eighths of the lanes idle.
#include <math.h>

#include <atomic>
#include <type_traits>

#include "pq_norm_row.h"

namespace pq {

namespace {

// ---- fast Hadamard transform of one row held in LDS as fp32, by one wave -------------------
// H = S_{2^k} (x) P_m / sqrt(K), channel i = a * m + b (a: Sylvester index, natural order; b: Paley
// index).  Kronecker factors act on separate index digits, so the transform is a sequence of
// passes, each applying a small matrix along one digit: every lane takes whole fibres (all elements
// that differ only in that digit), transforms them in registers and writes them back.  (The general path.)

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

// ---- the transform in registers: v[] are V values of a lane whose indices differ in the bits that name the register
// sums and differences of the registers that differ in bit S
template <int S, int V>
__device__ __forceinline__ void register_stage(float (&v)[V]) {
#pragma unroll
  for (int i = 0; i < V; ++i) {
    if (i & S) continue;
    const float a = v[i], b = v[i | S];
    v[i] = a + b;
    v[i | S] = a - b;
  }
}
// from bit S up to the last
template <int S, int V>
__device__ __forceinline__ void register_stages(float (&v)[V]) {
  if constexpr (S < V) {
    register_stage<S>(v);
    register_stages<2 * S>(v);
  }
}
// of the lanes that a DPP control word exchanges; sign: -1 in the lanes whose bit is set
template <int CTRL, int V>
__device__ __forceinline__ void lane_stage(float (&v)[V], float sign) {
#pragma unroll
  for (int i = 0; i < V; ++i) v[i] = dpp_f32<CTRL>(v[i]) + v[i] * sign;
}
// of the two halves of the wave (HALVES), or of the even and the odd rows of 16 lanes: a swap brings the partners of two
// registers into the same lanes, a second one takes the results back
template <bool HALVES, int V>
__device__ __forceinline__ void swap_stage(float (&v)[V]) {
  const auto swap = [](float& a, float& b) {
    const auto r = HALVES ? __builtin_amdgcn_permlane32_swap(as_u32(a), as_u32(b), false, false)
                          : __builtin_amdgcn_permlane16_swap(as_u32(a), as_u32(b), false, false);
    a = as_f32(r[0]);
    b = as_f32(r[1]);
  };
#pragma unroll
  for (int i = 0; i < V; i += 2) {
    swap(v[i], v[i + 1]);
    const float a = v[i], b = v[i + 1];
    v[i] = a + b;
    v[i + 1] = a - b;
    swap(v[i], v[i + 1]);
  }
}

typedef short bf16x4_bits __attribute__((ext_vector_type(4)));

// the non-zero squares modulo Q (Q prime), a bit each
template <int Q>
__host__ __device__ constexpr uint32_t squares() {
  uint32_t m = 0;
  for (int r = 1; r < Q; ++r)
    if (legendre<Q>(r) > 0) m |= 1u << r;
  return m;
}
// entry (b, n) of the Paley matrix of order M as bf16; zero outside of it, where the difference of the indices is no residue
template <int M>
__host__ __device__ constexpr uint32_t paley_bits(int b, int n) {
  constexpr uint32_t kSquares = squares<M - 1>();
  const int d = b - n + (b < n ? M - 1 : 0);
  const bool positive = b == n || b == 0 || (n != 0 && ((kSquares >> (d & 31)) & 1));
  return b < M && n < M ? (positive ? 0x3F80u : 0xBF80u) : 0u;
}
// every entry that a lane asks for; evaluated by the compiler, which refuses what the language leaves undefined
template <int M>
constexpr bool paley_bits_agree() {
  for (int b = 0; b < 32; ++b)
    for (int n = 0; n < 32; ++n)
      if (paley_bits<M>(b, n) != (b >= M || n >= M ? 0u : paley_entry<M>(b, n) > 0 ? 0x3F80u : 0xBF80u)) return false;
  return true;
}
static_assert(paley_bits_agree<12>() && paley_bits_agree<20>(), "the matrix of the matrix unit is the one of paley_pass");

// entries (b0 + 0 .. 3, n)
template <int M>
__device__ __forceinline__ bf16x4_bits paley_column4(int b0, int n) {
  uint32_t e[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) e[i] = paley_bits<M>(b0 + i, n);
  return __builtin_bit_cast(bf16x4_bits, make_uint2(e[0] | (e[1] << 16), e[2] | (e[3] << 16)));
}

// One row through a team of TEAM waves, V values a lane, into `slab` in the row's own order as bf16.  `slab_f` (a team of
// four): the row as fp32, for the last two bits of a, which are the wave's number.
template <int M, int V, int TEAM>
__device__ __forceinline__ void transform_row(const uint16_t* __restrict__ xr, float scale, uint16_t* slab, float* slab_f,
                                              int wave, int lane, int tl, int Ki) {
  float v[V];
  const int wv = TEAM == 1 ? 0 : wave;
  // lanes of m = 1: chunk of 8 channels `lane_chunk` of 64; the exchanges of lanes 1, 2, 7 and 8 apart (exclusive or) flip one
  // bit of it each
  const int lane_chunk = lane ^ ((lane & 4) ? 3 : 0);
  const int n = M == 12 ? lane & 15 : lane & 31;             // m = 12, 20: the Paley index
  const int j = M == 12 ? lane >> 4 : lane >> 5;
  if constexpr (M == 1) {
    uint4 lines[V / 8];
#pragma unroll
    for (int t = 0; t < V / 8; ++t)
      lines[t] = *reinterpret_cast<const uint4*>(xr + ((wv * (V / 8) + t) * 64 + lane_chunk) * 8);
#pragma unroll
    for (int t = 0; t < V / 8; ++t) {
      const uint32_t d[4] = {lines[t].x, lines[t].y, lines[t].z, lines[t].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[8 * t + 2 * e] = bf16_lo(d[e]);
        v[8 * t + 2 * e + 1] = bf16_hi(d[e]);
      }
    }
    register_stage<1>(v);
    register_stage<2>(v);
    register_stage<4>(v);
    const auto sign = [&](int bit) { return as_f32(0x3F800000u | (((uint32_t)lane_chunk >> bit & 1u) << 31)); };
    lane_stage<0xB1>(v, sign(0));                            // lane ^ 1
    lane_stage<0x4E>(v, sign(1));                            // lane ^ 2
    lane_stage<0x141>(v, sign(2));                           // lane ^ 7
    lane_stage<0x128>(v, sign(3));                           // lane ^ 8
    swap_stage<false>(v);
    swap_stage<true>(v);
    register_stages<8>(v);
  } else if constexpr (M == 12) {
    // sixteen fibres (16 x 12 contiguous values) times P_12 padded to 16 x 16 is one v_mfma_f32_16x16x16_bf16: lane l holds
    // A[l % 16][4 (l / 16) + i] (a fibre's values 4j .. 4j + 3: eight contiguous bytes), B[4 (l / 16) + i][l % 16] and
    // D[4 (l / 16) + i][l % 16].  Inputs and entries are exact in bf16, the products are accumulated in fp32.
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    const bf16x4_bits b = paley_column4<12>(4 * j, n);
    uint2 a[V / 4];
#pragma unroll
    for (int g = 0; g < V / 4; ++g) {
      a[g] = make_uint2(0u, 0u);
      if (j < 3) a[g] = *reinterpret_cast<const uint2*>(xr + ((wv * (V / 4) + g) * 16 + n) * 12 + 4 * j);
    }
#pragma unroll
    for (int g = 0; g < V / 4; ++g) {
      const f32x4 d = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(bf16x4_bits, a[g]), b,
                                                                (f32x4){0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[4 * g + i] = d[i];
    }
    register_stage<1>(v);
    register_stage<2>(v);
    swap_stage<false>(v);
    swap_stage<true>(v);
    register_stages<4>(v);
  } else {
    // 32 fibres times P_20 padded to 24 x 32, three v_mfma_f32_32x32x8_bf16: lane l holds A[l % 32][4 (l / 32) + i],
    // B[4 (l / 32) + i][l % 32] and D[8 (r / 4) + 4 (l / 32) + r % 4][l % 32]
    typedef float f32x16 __attribute__((ext_vector_type(16)));
    const bf16x4_bits b0 = paley_column4<20>(4 * j, n), b1 = paley_column4<20>(8 + 4 * j, n), b2 = paley_column4<20>(16 + 4 * j, n);
    uint2 a[V / 16][3];
#pragma unroll
    for (int g = 0; g < V / 16; ++g) {
      const uint16_t* f = xr + ((wv * (V / 16) + g) * 32 + n) * 20 + 4 * j;
      a[g][0] = *reinterpret_cast<const uint2*>(f);
      a[g][1] = *reinterpret_cast<const uint2*>(f + 8);
      a[g][2] = make_uint2(0u, 0u);
      if (j == 0) a[g][2] = *reinterpret_cast<const uint2*>(f + 16);
    }
#pragma unroll
    for (int g = 0; g < V / 16; ++g) {
      f32x16 d = {};
      d = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(__builtin_bit_cast(bf16x4_bits, a[g][0]), b0, d, 0, 0, 0);
      d = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(__builtin_bit_cast(bf16x4_bits, a[g][1]), b1, d, 0, 0, 0);
      d = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(__builtin_bit_cast(bf16x4_bits, a[g][2]), b2, d, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 16; ++r) v[16 * g + r] = d[r];
    }
    register_stage<1>(v);
    register_stage<2>(v);
    swap_stage<true>(v);
    register_stages<4>(v);
  }
  // channel of register i, for m = 12, 20
  const auto channel = [&](int i) {
    const int a = M == 12 ? (wv * (V / 4) + i / 4) * 16 + 4 * j + i % 4
                          : (wv * (V / 16) + i / 16) * 32 + 8 * (i % 16 / 4) + 4 * j + i % 4;
    return a * M + n;
  };
  if constexpr (TEAM == 1) {
    if constexpr (M == 1) {
#pragma unroll
      for (int t = 0; t < V / 8; ++t) {
        uint32_t d[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) d[e] = pack_bf16_rne(v[8 * t + 2 * e] * scale, v[8 * t + 2 * e + 1] * scale);
        *reinterpret_cast<uint4*>(slab + (t * 64 + lane_chunk) * 8) = make_uint4(d[0], d[1], d[2], d[3]);
      }
    } else if (n < M) {
#pragma unroll
      for (int i = 0; i < V; i += 2) {
        const uint32_t two = pack_bf16_rne(v[i] * scale, v[i + 1] * scale);
        slab[channel(i)] = (uint16_t)two;
        slab[channel(i + 1)] = (uint16_t)(two >> 16);
      }
    }
  } else {
    if constexpr (M == 1) {
#pragma unroll
      for (int t = 0; t < V / 8; ++t) {
        float4* out = reinterpret_cast<float4*>(slab_f + ((wv * (V / 8) + t) * 64 + lane_chunk) * 8);
        out[0] = make_float4(v[8 * t], v[8 * t + 1], v[8 * t + 2], v[8 * t + 3]);
        out[1] = make_float4(v[8 * t + 4], v[8 * t + 5], v[8 * t + 6], v[8 * t + 7]);
      }
    } else if (n < M) {
#pragma unroll
      for (int i = 0; i < V; ++i) slab_f[channel(i)] = v[i];
    }
    __syncthreads();
    // four channels of each quarter of the row
    const int quarter = Ki / 4;
    for (int q = tl * 4; q < quarter; q += 64 * TEAM * 4) {
      float w[4][4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const float4 f = *reinterpret_cast<const float4*>(slab_f + t * quarter + q);
        w[0][t] = f.x;
        w[1][t] = f.y;
        w[2][t] = f.z;
        w[3][t] = f.w;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) register_stages<1>(w[e]);
#pragma unroll
      for (int t = 0; t < 4; ++t)
        *reinterpret_cast<uint2*>(slab + t * quarter + q) = make_uint2(pack_bf16_rne(w[0][t] * scale, w[1][t] * scale),
                                                                       pack_bf16_rne(w[2][t] * scale, w[3][t] * scale));
    }
  }
  team_sync<TEAM>();
}

struct HadamardArgs {
  const int32_t* perm;          // pi, or null for the identity
  uint16_t* y;                  // bf16 [rows][ldy] rotated, reordered output, or null
  int64_t ldy;
  int pow2, m;                  // K = pow2 * m, m in {1, 12, 20}
  float scale;                  // 1 / sqrt(K)
};

// values a lane holds when `team` waves take a row
__host__ __device__ constexpr int lane_values(int64_t K, int m, int team) { return (int)(K / ((m == 1 ? 64 : m == 12 ? 48 : 40) * team)); }

// M: the Paley order of the row in registers, or 0: the general path.  WIDE: 64 values a lane, otherwise up to 32
template <int FMT, int G, int TEAM, int M, bool WIDE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WIDE ? 4 : 5))) void hadamard_rows_kernel(
    const uint16_t* __restrict__ x, int64_t rows, int64_t K, int64_t ld, const float* __restrict__ tensor_scale,
    int64_t steps, int64_t units, uint8_t* __restrict__ p_codes, uint16_t* __restrict__ p_scales,
    float* __restrict__ p_mul, HadamardArgs ha) {
  constexpr bool IS_INT = FMT == kInt4 || FMT == kInt3;
  // dynamic LDS: [per team: K fp32 (general path), K bf16 (one wave) or K fp32 and K bf16 (four)]
  //              [per team, INT: `units` fp32 group maxima] [per wave: 4 floats for team reductions]
  constexpr int kSlabBytes = M == 0 ? 4 : TEAM == 1 ? 2 : 6;
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
  em.y = ha.y;
  em.ldy = ha.ldy;
  em.T = em.encT = 0.0f;
  em.scale = ha.scale;
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
  constexpr int kBatch = 3;
  if constexpr (M == 0) {
    float* slab_f = reinterpret_cast<float*>(slab);
    constexpr int kInFlight = 8;
    const bool paley_on_mfma = ha.m == 12 && ha.pow2 >= 16;      // uniform
    if (paley_on_mfma) paley12_pass_from_memory<TEAM>(xr, slab_f, ha.pow2, tl);
    for (int c0 = 0; c0 < (paley_on_mfma ? 0 : k_chunks); c0 += kInFlight * 64 * TEAM) {
      uint4 lines[kInFlight];
#pragma unroll
      for (int t = 0; t < kInFlight; ++t) {
        const int c = min(c0 + t * 64 * TEAM + tl, k_chunks - 1);
        lines[t] = *reinterpret_cast<const uint4*>(xr + (size_t)c * 8);
      }
#pragma unroll
      for (int t = 0; t < kInFlight; ++t) {
        const int c = c0 + t * 64 * TEAM + tl;
        if (c < k_chunks) {
          const uint4 p = lines[t];
          *reinterpret_cast<float4*>(slab_f + c * 8) = make_float4(bf16_lo(p.x), bf16_hi(p.x), bf16_lo(p.y), bf16_hi(p.y));
          *reinterpret_cast<float4*>(slab_f + c * 8 + 4) = make_float4(bf16_lo(p.z), bf16_hi(p.z), bf16_lo(p.w), bf16_hi(p.w));
        }
      }
    }
    team_sync<TEAM>();
    hadamard_row<TEAM>(slab_f, Ki, ha.pow2, ha.m, tl, paley_on_mfma);
    Idx8 ix[kBatch];
#pragma unroll
    for (int q = 0; q < kBatch; ++q) ix[q] = load_idx(ha.perm, tl + 64 * TEAM * q, k_chunks);
    emit_row<FMT, G, TEAM, true>(slab_f, ha.perm, ix, em);
  } else {
    float* slab_f = reinterpret_cast<float*>(slab);          // a team of four: before the bf16 row
    uint16_t* slab_b = reinterpret_cast<uint16_t*>(slab + (TEAM == 1 ? 0 : (size_t)Ki * 4));
    const auto transform = [&](auto v) {
      transform_row<M, decltype(v)::value, TEAM>(xr, ha.scale, slab_b, slab_f, wave, lane, tl, Ki);
    };
    if constexpr (WIDE) {
      transform(std::integral_constant<int, 64>());
    } else {
      const int values = lane_values(K, M, TEAM);            // uniform
      if (values == 32) transform(std::integral_constant<int, 32>());
      else if (values == 16) transform(std::integral_constant<int, 16>());
      else if constexpr (M != 20) transform(std::integral_constant<int, 8>());
    }
    Idx8 ix[kBatch];
#pragma unroll
    for (int q = 0; q < kBatch; ++q) ix[q] = load_idx(ha.perm, tl + 64 * TEAM * q, k_chunks);
    emit_row<FMT, G, TEAM, false>(slab_b, ha.perm, ix, em);
  }
}

template <int FMT, int G, int TEAM, int M, bool WIDE>
int launch_hadamard_team(const void* x, int64_t rows, int64_t K, int64_t ld, const float* ts, const OperandLayout& L,
                         uint8_t* operand, const HadamardArgs& ha, hipStream_t st) {
  constexpr bool is_int = FMT == kInt4 || FMT == kInt3;
  auto kern = hadamard_rows_kernel<FMT, G, TEAM, M, WIDE>;
  // rows of a wave each: four a workgroup write more of a line together, one spreads few rows best (general path, reorder
  // alone: 1250 x 256 four a workgroup 4.5 us, one 4.1)
  const int n_waves = TEAM > 1 ? TEAM : rows > (M == 0 ? 1536 : 1024) ? 4 : 1;
  const int teams = TEAM == 1 ? n_waves : 1;
  const size_t shmem = (size_t)teams * (K * (M == 0 ? 4 : TEAM == 1 ? 2 : 6) + (is_int ? L.units * 4 : 0)) + (size_t)n_waves * 16;
  static std::atomic<uint64_t> raised{0};
  if (shmem > 48 * 1024) {
    if (int rc = allow_lds(reinterpret_cast<const void*>(kern), kNormLdsLimit, raised, "hipFuncSetAttribute(hadamard_rows_kernel)"))
      return rc;
  }
  const int64_t groups = (rows + teams - 1) / teams;
  hipLaunchKernelGGL(kern, dim3((unsigned)groups), dim3(64 * n_waves), shmem, st, (const uint16_t*)x, rows, K, ld, ts,
                     L.steps, L.units, operand ? operand + L.codes : nullptr,
                     (uint16_t*)(operand ? operand + L.scales : nullptr),
                     (float*)(operand ? operand + L.mul : nullptr), ha);
  return check_hip(hipGetLastError(), "hadamard_rows_kernel");
}

// Whether four waves share a row that one could hold: with few rows its chain is what takes the time, with many the exchange
// through LDS is.  One wave and four, us, NVFP4: 512 x 1536 4.9, 4.0; 1024 x 1536 5.0, 5.1; 1536 x 2048 7.2, 6.5; 2048 x 2048
// 7.4, 7.9; 1536 x 2560 8.8, 8.8; 1536 x 3072 9.7, 8.7; 2048 x 3072 10.1, 10.4; 4608 x 4096 24.1, 21.5; 8192 x 4096 34.0, 35.3.
bool hadamard_four_waves(int64_t rows, int64_t K) {
  return K >= 4096 ? rows <= 6144 : K >= 2048 ? rows <= 1536 : K >= 1536 && rows <= 768;
}

template <int FMT, int G>
int launch_hadamard(const void* x, int64_t rows, int64_t K, int64_t ld, const float* ts, const OperandLayout& L,
                    uint8_t* operand, const HadamardArgs& ha, hipStream_t st) {
  // the widths that are taken: an fp32 row and the group maxima in LDS
  constexpr bool is_int = FMT == kInt4 || FMT == kInt3;
  const size_t least = (size_t)K * 4 + (is_int ? L.units * 4 : 0) + (size_t)(K > 4096 ? 4 : 1) * 16;
  if (least > kNormLdsLimit)
    return fail(PQ_ERR_SHAPE, "K=%lld needs %zu bytes of LDS for one row and the vectors, more than the %zu available",
                (long long)K, least, kNormLdsLimit);
  const auto in_registers = [&](int team) {
    const int v = lane_values(K, ha.m, team);
    return (v == 8 && ha.m != 20) || v == 16 || v == 32 || v == 64;
  };
  bool four = hadamard_four_waves(rows, K);
  if (!in_registers(four ? 4 : 1)) four = in_registers(4) || !(in_registers(1) || K <= 4096);
  if (rows * 256 > UINT32_MAX) four = false;                  // more threads than a grid holds
  const bool wide = lane_values(K, ha.m, four ? 4 : 1) == 64;
#define PQ_HADAMARD(TEAM, M, WIDE) return launch_hadamard_team<FMT, G, TEAM, M, WIDE>(x, rows, K, ld, ts, L, operand, ha, st)
#define PQ_HADAMARD_M(M)                              \
  if (four && wide) PQ_HADAMARD(4, M, true);          \
  if (four) PQ_HADAMARD(4, M, false);                 \
  if (wide) PQ_HADAMARD(1, M, true);                  \
  PQ_HADAMARD(1, M, false)
  if (!in_registers(four ? 4 : 1)) {
    if (four) PQ_HADAMARD(4, 0, false);
    PQ_HADAMARD(1, 0, false);
  }
  switch (ha.m) {
    case 1: PQ_HADAMARD_M(1);
    case 12: PQ_HADAMARD_M(12);
    default: PQ_HADAMARD_M(20);
  }
#undef PQ_HADAMARD_M
#undef PQ_HADAMARD
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

HadamardArgs hadamard_args(const int32_t* perm, int64_t K, void* y, int64_t ldy, int pow2, int m) {
  HadamardArgs na = {};
  na.perm = perm;
  na.y = (uint16_t*)y;
  na.ldy = ldy;
  na.pow2 = pow2;
  na.m = m;
  na.scale = (float)(1.0 / sqrt((double)K));
  return na;
}

}  // namespace

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
  return launch_hadamard<kFmtNone, 64>(x, rows, K, ld, nullptr, L, nullptr, hadamard_args(perm, K, y, ldy, p, m), st);
}

int run_hadamard_quantize_packed(const int32_t* perm, pq_format fmt, int group, const void* x, int64_t rows,
                                 int64_t K, int64_t ld, const float* ts, void* operand, void* y, int64_t ldy,
                                 hipStream_t st) {
  int p, m;
  if (!hadamard_factor(K, &p, &m)) return fail(PQ_ERR_SHAPE, "no Hadamard construction for K=%lld", (long long)K);
  const OperandLayout L = operand_layout(fmt, group, rows, K);
  const HadamardArgs na = hadamard_args(perm, K, y, ldy, p, m);
  uint8_t* o = (uint8_t*)operand;
  if (fmt == PQ_FMT_NVFP4) return launch_hadamard<kNvfp4, 16>(x, rows, K, ld, ts, L, o, na, st);
#define PQ_INT_CASE(F, FE)                                                           \
  if (fmt == F) {                                                                    \
    switch (group) {                                                                 \
      case 32: return launch_hadamard<FE, 32>(x, rows, K, ld, ts, L, o, na, st);   \
      case 64: return launch_hadamard<FE, 64>(x, rows, K, ld, ts, L, o, na, st);   \
      case 128: return launch_hadamard<FE, 128>(x, rows, K, ld, ts, L, o, na, st); \
      case 256: return launch_hadamard<FE, 256>(x, rows, K, ld, ts, L, o, na, st); \
    }                                                                                \
  }
  PQ_INT_CASE(PQ_FMT_INT4, kInt4)
  PQ_INT_CASE(PQ_FMT_INT3, kInt3)
#undef PQ_INT_CASE
  return fail(PQ_ERR_FORMAT, "unsupported (format, group) = (%d, %d)", (int)fmt, group);
}

}  // namespace pq
