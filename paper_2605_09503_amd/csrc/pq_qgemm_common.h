// Operand slices of the qgemm kernel, their loading and exact unpacking to scaled fp16 (see
// pq_qgemm.hip for why fp16 operands carry the per-group scales exactly).
#pragma once
#include <type_traits>

#include "pq_device.h"
#include "pq_host.h"

namespace pq {

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float16_t __attribute__((ext_vector_type(16)));

constexpr int kBK = 64;                 // K elements per step
constexpr int kRowBytes = kBK * 2 + 16; // fp16 row in LDS, padded by one 16-byte piece: with 144-byte
                                        // rows both the 16-byte fragment reads (rows 0..31 of a
                                        // piece) and the unpack writes spread over all banks

__device__ __forceinline__ half2_t as_h2(uint32_t u) { return __builtin_bit_cast(half2_t, u); }
__device__ __forceinline__ uint32_t h2_bits(half2_t h) { return __builtin_bit_cast(uint32_t, h); }

// ------------------------------------------------------------------------ operand unpack
// Per-thread slice of a tile row: 32 consecutive k (16 bytes of codes) plus its scales.
struct Slice {
  uint4 codes;
  uint32_t sc;      // NVFP4: two E4M3 bytes (k 0-15, 16-31); INT: one fp16 in the low half
};

// Where a quantized operand lives.  One description covers both layouts the kernel reads:
//   codes of (row, K step, half)  at codes  + row * code_row + step * code_step + half * 16
//   scale unit u of a row         at scales + row * sc_row   + u * sc_step          (2 bytes)
// where a scale unit is the pair of E4M3 bytes of 32 consecutive k (NVFP4, u = k / 32) or the
// fp16 normalised maximum of a group (INT, u = k / G).
//   row-major (as the quantizers store it): code_row = K / 2, code_step = 32;
//                                           sc_row = K / 16 (NVFP4) or 2 K / G, sc_step = 2
//   panel (K-step-major, see pq_pack.hip):  code_row = 32, code_step = 32 * rows;
//                                           sc_row = 2, sc_step = 2 * rows
// mul: per-row epilogue factor (stride 1) or a single factor (stride 0).
// panel: the panel layout.  marked: the sign of a row's factor says that the row holds INT3 codes beyond three bits
// (always in the panel layout; set by the scale preparation of a row-major operand when it sees the codes)
// bias: bf16 value per row of this operand added to the product in the epilogue (used for the
// weight operand, whose rows are the output columns), or null.
struct OperandView {
  const uint8_t* codes;
  int64_t code_row;
  int code_step;
  const uint8_t* scales;
  int64_t sc_row;
  int sc_step;
  const float* mul;
  int mul_stride;
  bool panel = false, marked = false;
  const uint16_t* bias = nullptr;
};

// Scale pair(s) handed to unpack_pair.  INT carries {h, h} and {-8 h, -8 h} (see below).
struct PairScale {
  half2_t mul, add;
};

// {s, s} pairs of the two group scales a slice can touch; all zero when it lies beyond K (ok is false), so that
// whatever codes were loaded contribute 0
template <int FMT>
__device__ __forceinline__ void slice_scales(const Slice& s, bool ok, PairScale& p0, PairScale& p1) {
  if constexpr (FMT == kNvfp4) {
    // E4M3 byte b -> fp16: bits (b << 7) read as fp16 are value * 2^-8, subnormals included
    uint32_t two = __builtin_amdgcn_perm(0u, s.sc, 0x0C010C00u) << 7;
    two = ok ? two : 0u;
    half2_t v = as_h2(two) * (half2_t){(_Float16)256.0f, (_Float16)256.0f};
    p0.mul = (half2_t){v.x, v.x};
    p1.mul = (half2_t){v.y, v.y};
    p0.add = p1.add = (half2_t){(_Float16)0.0f, (_Float16)0.0f};
  } else {
    uint32_t b = (s.sc & 0xFFFFu) | (s.sc << 16);
    half2_t v = as_h2(ok ? b : 0u);
    p0.mul = p1.mul = v;
    p0.add = p1.add = v * (half2_t){(_Float16)-8.0f, (_Float16)-8.0f};
  }
}

// two codes of dword d (pair j of four: bytes 2 (j % 2) and the next of the low, j < 2, or high nibbles for INT, byte j for
// NVFP4) -> two scaled fp16 values.  Which two elements form a pair only has to be the same for A and W.
//
// INT: the two's complement nibble z becomes offset binary u = z + 8 (flip bit 3) in a byte of its own, which as E4M3 is u 2^-9
// (subnormals and the first binade are linear); the conversion unit makes two of them fp16 u, and one fused multiply-add forms
// u h - 8 h = z h.  u h has at most 12 significant bits, 8 h has 8, the result 11: every step is exact in the fma.  11
// instructions for eight codes; with each nibble shifted into the mantissa of a constant 12: INT4 g64 2048 x 3072 x 3072 41.7 ->
// 40.1 us, 512 x 9216 x 3072 31.9 -> 30.8, g32 4608 x 3072 x 3072 76.8 -> 75.2, INT3 g32 8192 x 12288 x 3072 463 -> 459.
template <int FMT, int J>
__device__ __forceinline__ uint32_t unpack_pair(uint32_t d, const PairScale& sc) {
  if constexpr (FMT == kNvfp4) {
    return h2_bits(__builtin_amdgcn_cvt_scalef32_pk_f16_fp4(d, 1.0f, J) * sc.mul);
  } else {
    const uint32_t x = ((J & 2 ? d >> 4 : d) & 0x0F0F0F0Fu) ^ 0x08080808u;
    const half2_t t = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8((int)x, 512.0f, J & 1);
    return h2_bits(__builtin_elementwise_fma(t, sc.mul, sc.add));
  }
}

// tile row `r`, 16-byte piece `piece` (0..7) -> byte offset inside one LDS operand tile
__device__ __forceinline__ int lds_off(int r, int piece) { return r * kRowBytes + (piece << 4); }

// ------------------------------------------------------------------------ codes for the matrix unit
// (pq_qgemm_group.hip says why these are exact)
typedef int int4v __attribute__((ext_vector_type(4)));
typedef int int8v __attribute__((ext_vector_type(8)));
typedef _Float16 half4v __attribute__((ext_vector_type(4)));

// four two's complement nibbles, one per byte of n (top nibbles 0), m = their sign bits: bytes sign << 7 | |z|
__device__ __forceinline__ uint32_t e4m3_bytes(uint32_t n, uint32_t m) {
  const uint32_t f = __builtin_amdgcn_perm(0u, 0x00008F00u, m);      // 0x8F where negative
  return (n ^ f) + m;                                                // 16 - n <= 8 under the sign: no carry
}

// eight nibbles z (two's complement, |z| <= 4) -> eight nibbles sign << 3 | |z|
__device__ __forceinline__ uint32_t e2m1_nibbles(uint32_t d) {
  const uint32_t s = d & 0x88888888u, m = s >> 3;
  return (d ^ (s - m)) + m;
}

// 32 codes of a row -> the 32 E4M3 bytes of a lane's operand (any order of k, as long as it is the same for A and W)
__device__ __forceinline__ int8v e4m3_operand(const uint4& c) {
  const uint32_t d[4] = {c.x, c.y, c.z, c.w};
  int8v o;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    o[2 * e] = (int)e4m3_bytes(d[e] & 0x0F0F0F0Fu, (d[e] >> 3) & 0x01010101u);
    o[2 * e + 1] = (int)e4m3_bytes((d[e] >> 4) & 0x0F0F0F0Fu, (d[e] >> 7) & 0x01010101u);
  }
  return o;
}

// fp16 scale unit as the one non-zero k of an outer product's operand
__device__ __forceinline__ half4v scale_operand(uint32_t h) {
  return __builtin_bit_cast(half4v, make_uint2(h, 0u));
}

// two fp32 rounded to nearest even bf16, packed (v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t cvt_pk_bf16(float lo, float hi) {
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){lo, hi}, bf16x2_t));
}

template <int V>
struct IntC {
  static constexpr int value = V;
};

// ------------------------------------------------------------------------ tile assignment
// Consecutive workgroup ids land on different XCDs (8 of them, each with its own L2); give every XCD a
// contiguous range of tiles, and walk tiles in bands of 8 along M so that concurrently running workgroups
// share A and W strips.
__device__ __forceinline__ void assign_tile(int tiles_m, int tiles_n, int& tile_m, int& tile_n) {
  const int n_tiles = tiles_m * tiles_n;
  int pid = blockIdx.x;
  {
    // XCD x runs the workgroups with id % 8 == x: (n_tiles - x + 7) / 8 of them, which get the tiles
    // from x * (n_tiles / 8) + min(x, n_tiles % 8) on
    const int x = pid & 7, q8 = n_tiles >> 3, r8 = n_tiles & 7;
    pid = x * q8 + min(x, r8) + (pid >> 3);
  }
  constexpr int BAND = 8;
  const int band_sz = BAND * tiles_n;
  const int band = pid / band_sz;
  const int band_m0 = band * BAND;
  const int band_h = min(BAND, tiles_m - band_m0);
  const int in_band = pid - band * band_sz;
  tile_m = band_m0 + in_band % band_h;
  tile_n = in_band / band_h;
}

// ------------------------------------------------------------------------ epilogue
// What becomes of the product: rounded to bf16, stored in fp32, or compared with a reference -- then only the sum of
// (ref - product)^2 over a workgroup's tile is kept, in fp64 (each difference exact, the sum in a fixed order):
// y[tile] = or += that sum.
enum OutKind : int { kOutBf16 = 0, kOutF32 = 1, kOutDiff = 2 };
struct Output {
  int kind;
  void* y;              // bf16 or float [M, ldy]; kOutDiff: double [tiles]
  int64_t ldy;          // kOutDiff: of ref
  const float* ref;     // kOutDiff only
  bool add;             // kOutDiff only
};
// A launch that compares may hold several problems of one shape and one reference, problem z in blockIdx.y: its operands
// lie z * a_next and z * w_next bytes further on, its sums z * y_next.  Only the kernels that compare are handed these: the
// larger argument alone changes how many registers the compiler gives the others (see FEW in pq_qgemm_split.hip).
struct Outputs : Output {
  size_t a_next = 0, w_next = 0;
  int64_t y_next = 0;
  unsigned problems = 1;
};
// A product that prepares the scales of its row-major INT operands itself (RAW in pq_qgemm_split.hip): the scales are those of
// codes up to q, and what a launch of the preparation would leave in the workspace goes there, for pq_qgemm_run.
struct RawScales {
  float q;
  uint16_t *a_units, *w_units;
  float *a_mul, *w_mul;
};
struct RawOutput : Output {
  RawScales raw;
};
template <int OUT, bool RAW = false>
using KernelOutput = std::conditional_t<RAW, RawOutput, std::conditional_t<OUT == kOutDiff, Outputs, Output>>;
static_assert(sizeof(Output) == 40, "a larger argument has changed the registers of the 32 x 32 tiles");

// the operands and the sums of this workgroup's problem (a factor of stride 0 is a tensor scale, the same for all)
__device__ __forceinline__ void enter_problem(OperandView& A, OperandView& W, Outputs& out) {
  const size_t z = blockIdx.y;
  auto move = [&](OperandView& v, size_t by) {
    v.codes += by;
    v.scales += by;
    if (v.mul_stride) v.mul = reinterpret_cast<const float*>(reinterpret_cast<const char*>(v.mul) + by);
  };
  move(A, z * out.a_next);
  move(W, z * out.w_next);
  out.y = reinterpret_cast<double*>(out.y) + (int64_t)z * out.y_next;
}

// the sums of a workgroup's threads, in a fixed order, to y[tile] (called by all threads; red: free LDS)
__device__ __forceinline__ void store_diff(double d2, double* red, int threads, int tile, const Output& out) {
  d2 = wave_sum(d2);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = d2;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int w = 0; w < threads / 64; ++w) t += red[w];
    double* p = reinterpret_cast<double*>(out.y) + tile;
    *p = out.add ? *p + t : t;
  }
}

// The epilogue's factors.  A product's rows and columns have a factor each (INT) and the columns perhaps a bias; they are
// asked for at the start of the kernel and wait in LDS.  Loaded where they are used, one to four at a time, they were a chain
// of memory latencies after the last step: 3.3 to 4.2 us of a 256 x 256 tile's epilogue (clock stamps; a round of tiles is
// 80 us at K = 3072), and one for each strip of a split tile.  Kernel alone, us, before -> now: NVFP4 4608 x 9216 x 3072 214.9 -> 208.0,
// 512 x 9216 x 3072 32.3 -> 29.6, 1024 x 3072 x 3072 22.2 -> 20.1, 256 x 512 x 512 3.60 -> 3.27; INT4 g64 4608 x 3072 x 3072 68.1 ->
// 66.3; INT3 g32 8192 x 12288 x 3072 484 -> 472, g64 512 x 3072 x 3072 12.0 -> 10.8.  In LDS: BM factors of rows, BN of columns, BN
// biases.
template <int BM, int BN, int T, bool INT>
struct Factors {
  static_assert(BN <= T, "a bias a thread");
  static constexpr int N = INT ? (BM + BN + T - 1) / T : 0;
  float mul[N > 0 ? N : 1], bias = 0.0f;               // this thread's

  __device__ __forceinline__ void load(const OperandView& A, const OperandView& W, int M, int N_, int m0, int n0) {
    const int tid = threadIdx.x;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int at = i * T + tid;
      mul[i] = at < BM ? A.mul[min(m0 + at, M - 1)] : W.mul[min(n0 + min(at, BM + BN - 1) - BM, N_ - 1)];
    }
    if (W.bias) bias = bf16_to_f32(W.bias[min(n0 + min(tid, BN - 1), N_ - 1)]);
  }
  __device__ __forceinline__ void put(float* factors) const {
    const int tid = threadIdx.x;
#pragma unroll
    for (int i = 0; i < N; ++i)
      if ((i + 1) * T <= BM + BN || i * T + tid < BM + BN) factors[i * T + tid] = mul[i];
    if (BN == T || tid < BN) factors[BM + BN + tid] = bias;
  }
};
template <int BM, int BN>
constexpr size_t kFactorBytes = (BM + 2 * BN) * sizeof(float);

// ------------------------------------------------------------------------ INT3 codes beyond three bits
// The quantizers write INT3 codes of -3 .. 3, but a nibble holds -8 .. 7, and an operand with any of them is
// multiplied as it is (E2M1 holds neither 5 nor 7).  Packing, and on the row-major layout the scale preparation of
// pq_qgemm, marks the rows that hold such codes in the sign of their factor, which the kernels look at in the
// epilogue; pq_qgemm_run, whose preparation has not seen the codes, looks at every code.  A workgroup that finds one
// computes its tile again with E4M3 operands straight from memory, over what it stored.  The sums are those of the
// kernel that calls, in its order (KS shares of the steps; every factor that differs is a power of two), so rows
// without such codes keep their bits.  Groups are a multiple of 64.  The marks cost nothing that shows (INT3 g64
// 512 x 3072 x 3072 14.2 us with and without); the scale preparation that sets them takes 0.3 to 1 us longer (2.2 at
// 31 x 2337 x 12288; four of a lane's pieces of codes asked for at once instead of one: the same), and looking at every
// code takes 13 to 20 % of a split tile's time and 2 to 5 of a large one's.
enum WideTest : int { kWideNone = 0, kWideMarks = 1, kWideCodes = 2 };

// a code beyond three bits sets bit 3 of its nibble (its bits 3 and 2 differ)
constexpr uint32_t kWideBits = 0x88888888u;
__device__ __forceinline__ uint32_t wide_codes(uint32_t d) { return d ^ (d << 1); }

// the factors of a tile's rows and columns, or-ed over what a lane reads: every wave looks at all of them, so that none has
// to tell the others
template <int BM, int BN>
__device__ __forceinline__ uint32_t tile_marks(const float* factors) {
  uint32_t v = 0;
#pragma unroll
  for (int r = 0; r < BM + BN; r += 64) v |= as_u32(factors[min(r + (int)(threadIdx.x & 63), BM + BN - 1)]);
  return v;
}

// whether any thread of the workgroup met a wide code (called by all of them); flags: an int per wave of LDS that
// nothing else uses
template <int WAVES>
__device__ __forceinline__ bool any_wide(uint32_t wide, int* flags) {
  const int mine = __any((wide & kWideBits) != 0);
  if ((threadIdx.x & 63) == 0) flags[threadIdx.x >> 6] = mine;
  __syncthreads();
  int any = 0;
#pragma unroll
  for (int v = 0; v < WAVES; ++v) any |= flags[v];
  return __builtin_amdgcn_readfirstlane(any) != 0;
}

// RAW: fp32 scales; the factors of the tile's rows and columns, and behind them 2^-E, are in LDS
template <int BM, int BN, int WAVES, int KS, int OUT, bool RAW = false>
__device__ __forceinline__ void wide_codes_tile(const OperandView& A, const OperandView& W, int M, int N, int K,
                                                int g_shift, int m0, int n0, const KernelOutput<OUT, RAW>& out,
                                                const float* factors = nullptr) {
  static_assert(OUT != kOutDiff, "the selection quantizes its operands itself");
  const int lane = threadIdx.x & 63;
  const int row = lane & 31, half = lane >> 5;
  const int ksteps = K / kBK;
  const float16_t zero = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f,
                          0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
  for (int b = threadIdx.x >> 6; b < BM / 32 * (BN / 32); b += WAVES) {
    const int m = m0 + b % (BM / 32) * 32 + row, nb = n0 + b / (BM / 32) * 32;
    const int64_t ar = min(m, M - 1), wr = min(nb + row, N - 1);
    const uint8_t *ac = A.codes + ar * A.code_row + half * 16, *wc = W.codes + wr * W.code_row + half * 16;
    const uint8_t *as = A.scales + ar * A.sc_row, *ws = W.scales + wr * W.sc_row;
    const float* const downs = factors + kFactorBytes<BM, BN> / 4;
    auto unit_at = [&](const uint8_t* at, int local) -> uint32_t {
      if constexpr (RAW) return int_scale_unit(*reinterpret_cast<const float*>(at), out.raw.q, downs[local]);
      else return *reinterpret_cast<const uint16_t*>(at);
    };
    float16_t sum = zero;
#pragma unroll 1
    for (int ks = 0; ks < KS; ++ks) {
      float16_t acc = zero;
#pragma unroll 1
      for (int s = ks; s < ksteps; s += KS) {
        const int64_t unit = (s * kBK) >> g_shift;
        const uint4 a = *reinterpret_cast<const uint4*>(ac + (int64_t)s * A.code_step);
        const uint4 w = *reinterpret_cast<const uint4*>(wc + (int64_t)s * W.code_step);
        const uint32_t sa = unit_at(as + unit * A.sc_step, m - m0), sw = unit_at(ws + unit * W.sc_step, BM + nb - n0 + row);
        const float16_t sc = __builtin_amdgcn_mfma_f32_32x32x8f16(scale_operand(half == 0 ? sw : 0u), scale_operand(sa),
                                                                  zero, 0, 0, 0);
        const float16_t p = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(e4m3_operand(w), e4m3_operand(a), zero, 0, 0,
                                                                            0, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = __builtin_fmaf(p[r], sc[r], acc[r]);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) sum[r] = ks == 0 ? acc[r] : sum[r] + acc[r];
    }
    if (m >= M) continue;
    const float am = fabsf(RAW ? factors[m - m0] : A.mul[(int64_t)m * A.mul_stride]);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int n = nb + r / 4 * 8 + half * 4 + r % 4;
      if (n >= N) continue;
      float v = (sum[r] * 262144.0f) * (am * fabsf(RAW ? factors[BM + n - n0] : W.mul[(int64_t)n * W.mul_stride]));
      if (W.bias) v += bf16_to_f32(W.bias[n]);
      if constexpr (OUT == kOutF32)
        reinterpret_cast<float*>(out.y)[(int64_t)m * out.ldy + n] = v;
      else
        reinterpret_cast<uint16_t*>(out.y)[(int64_t)m * out.ldy + n] = (uint16_t)cvt_pk_bf16(v, 0.0f);
    }
  }
}

// The accumulators of a workgroup's output tile, scaled and stored.  unit: a power of two that undoes the
// operands' fixed code scale (1 where they have none; the product with it is exact).  factors: as Factors left them
// (INT: magnitudes, their sign a mark); NVFP4 has one factor for all, nv_mul, the product of its tensor scales.
template <int BM, int BN, int WTM, int WTN, int TM, int TN, bool RAGGED_M, int T, int SMEM_BYTES, int OUT, bool INT, bool BIAS>
__device__ __forceinline__ void store_tile_as(const float16_t (&acc)[TN][TM], unsigned char* smem, const float* factors,
                                              float nv_mul, int M, int N, int m0, int n0, int wave_m, int wave_n, int tm_cnt,
                                              int tid, float unit, int tile, const Output& out) {
  void* __restrict__ y = out.y;
  const int64_t ldy = out.ldy;
  double d2 = 0.0;
  const int lane = tid & 63;
  const int frag_row = lane & 31, frag_half = lane >> 5;
  // A lane holds, per MFMA tile, column m = lane % 32 and rows
  // n = 8 * (r / 4) + 4 * (lane / 32) + r % 4.  The bf16 tile is staged through LDS (the
  // operand stages are free after the last barrier) so that global stores are 16 bytes per
  // lane and contiguous along n; the fp32 variant (a checking aid) stores directly.
  constexpr int C_ROW_BYTES = BN * 2 + 16;
  static_assert(OUT != kOutBf16 || BM * C_ROW_BYTES <= SMEM_BYTES, "output tile fits in the operand stages");
  // The column factors (and the optional bias of the linear layer, y = x W^T + b) do not depend on
  // the row block: read once (16 per MFMA tile column).
  float wm[INT ? TN : 1][16], wb[BIAS ? TN : 1][16];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float* at = factors + BM + wave_n * WTN + i * 32 + q * 8 + frag_half * 4;
      if constexpr (INT) {
        const float4 f = *reinterpret_cast<const float4*>(at);
        wm[i][q * 4] = fabsf(f.x); wm[i][q * 4 + 1] = fabsf(f.y); wm[i][q * 4 + 2] = fabsf(f.z); wm[i][q * 4 + 3] = fabsf(f.w);
      }
      if constexpr (BIAS) {
        const float4 f = *reinterpret_cast<const float4*>(at + BN);
        wb[i][q * 4] = f.x; wb[i][q * 4 + 1] = f.y; wb[i][q * 4 + 2] = f.z; wb[i][q * 4 + 3] = f.w;
      }
    }
  float am[TM];
#pragma unroll
  for (int j = 0; j < TM; ++j) {
    am[j] = 0.0f;
    if constexpr (INT)
      if (!RAGGED_M || j < tm_cnt) am[j] = fabsf(factors[wave_m * WTM + j * 32 + frag_row]);
  }
#pragma unroll
  for (int j = 0; j < TM; ++j) {
    if (RAGGED_M && j >= tm_cnt) break;         // wave-uniform
    const int ml = wave_m * WTM + j * 32 + frag_row;
    const int m = m0 + ml;
#pragma unroll
    for (int i = 0; i < TN; ++i) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int nl = wave_n * WTN + i * 32 + q * 8 + frag_half * 4;
        const int n = n0 + nl;
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[e] = (acc[i][j][q * 4 + e] * unit) * (INT ? am[j] * wm[INT ? i : 0][q * 4 + e] : nv_mul);
          if constexpr (BIAS) v[e] += wb[BIAS ? i : 0][q * 4 + e];
        }
        if constexpr (OUT == kOutDiff) {
          if (m < M && n < N) {
            const float* r = out.ref + (int64_t)m * ldy + n;
            float f[4];
            if (n + 3 < N) {
              const float4 whole = *reinterpret_cast<const float4*>(r);
              f[0] = whole.x; f[1] = whole.y; f[2] = whole.z; f[3] = whole.w;
            } else {
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                f[e] = n + e < N ? r[e] : 0.0f;
                v[e] = n + e < N ? v[e] : 0.0f;        // no column: no difference
              }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const double d = (double)f[e] - (double)v[e];
              d2 = fma(d, d, d2);
            }
          }
        } else if constexpr (OUT == kOutF32) {
          if (m < M && n < N) {
            float* yo = reinterpret_cast<float*>(y) + (int64_t)m * ldy + n;
            if (n + 3 < N) {
              *reinterpret_cast<float4*>(yo) = make_float4(v[0], v[1], v[2], v[3]);
            } else {
              for (int e = 0; e < 4 && n + e < N; ++e) yo[e] = v[e];
            }
          }
        } else {
          *reinterpret_cast<uint2*>(smem + ml * C_ROW_BYTES + nl * 2) =
              make_uint2(cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3]));
        }
      }
    }
  }
  if constexpr (OUT == kOutDiff) store_diff(d2, reinterpret_cast<double*>(smem), T, tile, out);
  if constexpr (OUT == kOutBf16) {
    __syncthreads();
    constexpr int CHUNKS_PER_ROW = BN / 8;               // 16-byte chunks of 8 bf16
    uint16_t* yb = reinterpret_cast<uint16_t*>(y);
#pragma unroll 4
    for (int c = tid; c < BM * CHUNKS_PER_ROW; c += T) {
      const int row = c / CHUNKS_PER_ROW, cc = c % CHUNKS_PER_ROW;
      const int m = m0 + row, n = n0 + cc * 8;
      if (m >= M || n >= N) continue;
      const uint4 v = *reinterpret_cast<const uint4*>(smem + row * C_ROW_BYTES + cc * 16);
      uint16_t* yo = yb + (int64_t)m * ldy + n;
      if (n + 7 < N) {
        // the output is not read again by this kernel: a streaming store keeps it from displacing
        // the operand strips in L2
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        __builtin_nontemporal_store((u32x4){v.x, v.y, v.z, v.w}, reinterpret_cast<u32x4*>(yo));
      } else {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
        for (int e = 0; e < 8 && n + e < N; ++e) yo[e] = (uint16_t)(w[e >> 1] >> (16 * (e & 1)));
      }
    }
  }
}

template <int BM, int BN, int WTM, int WTN, int TM, int TN, bool RAGGED_M, int T, int SMEM_BYTES, int OUT, bool INT>
__device__ __forceinline__ void store_tile(const float16_t (&acc)[TN][TM], unsigned char* smem, const float* factors,
                                           float nv_mul, bool bias, int M, int N, int m0, int n0, int wave_m, int wave_n,
                                           int tm_cnt, int tid, float unit, int tile, const Output& out) {
  // without a bias the product is stored as it is (a -0 stays -0)
  if (OUT != kOutDiff && bias)
    store_tile_as<BM, BN, WTM, WTN, TM, TN, RAGGED_M, T, SMEM_BYTES, OUT, INT, true>(acc, smem, factors, nv_mul, M, N, m0, n0,
                                                                                     wave_m, wave_n, tm_cnt, tid, unit, tile, out);
  else
    store_tile_as<BM, BN, WTM, WTN, TM, TN, RAGGED_M, T, SMEM_BYTES, OUT, INT, false>(acc, smem, factors, nv_mul, M, N, m0, n0,
                                                                                      wave_m, wave_n, tm_cnt, tid, unit, tile, out);
}

// view of an operand in the panel layout (pq_pack.hip)
inline OperandView panel_view(pq_format fmt, int group, const void* operand, int64_t rows, int64_t K,
                              const float* tensor_scale) {
  const OperandLayout L = operand_layout(fmt, group, rows, K);
  const uint8_t* o = (const uint8_t*)operand;
  OperandView v;
  v.panel = v.marked = true;
  v.codes = o + L.codes;
  v.code_row = 32;
  v.code_step = (int)(rows * 32);
  v.scales = o + L.scales;
  v.sc_row = 2;
  v.sc_step = (int)(rows * 2);
  if (fmt == PQ_FMT_NVFP4) {
    v.mul = tensor_scale;
    v.mul_stride = 0;
  } else {
    v.mul = (const float*)(o + L.mul);
    v.mul_stride = 1;
  }
  return v;
}

// the product kernel on two operand views (pq_qgemm.hip), with the given tile
int launch_qgemm_views(pq_format fmt, int group, const OperandView& A, const OperandView& W, int64_t M,
                       int64_t N, int64_t K, const Outputs& out, int tile, hipStream_t st);
// tiles (= workgroups) of that launch
int64_t qgemm_tiles(int tile, int64_t M, int64_t N);
// output tiles of the product kernels (choose_tile in pq_qgemm_tile.hip)
enum Tile : int { kTile256 = 1, kTile128 = 2, kTile224 = 3, kTileSplit32 = 4, kTileSplit64x32 = 5, kTileSplit64 = 6, kTileSplit64x96 = 7,
                  kTileSplit64Eight = 8, kTileSplit64x96Eight = 9 };     // the same two with eight waves
// small outputs (pq_qgemm_split.hip)
int launch_qgemm_split(pq_format fmt, int group, const OperandView& A, const OperandView& W, int M, int N, int K,
                       const Outputs& out, int tile, hipStream_t st);
// whether a product of row-major INT operands prepares their scales in the product kernel, and that product
bool split_takes_raw_scales(pq_format fmt, int group, int tile, int64_t M, int64_t N, int64_t K);
int launch_qgemm_split_raw(pq_format fmt, int group, const OperandView& A, const OperandView& W, int M, int N, int K,
                           const RawOutput& out, int tile, hipStream_t st);
// the integer formats' large outputs with groups of 64 and more (pq_qgemm_group.hip)
int launch_qgemm_group(pq_format fmt, int group, const OperandView& A, const OperandView& W, int M, int N, int K,
                       const Outputs& out, int tile, hipStream_t st);

}  // namespace pq
