// Low-bit GEMM of the quantized layer (paper Eq. 8) for outputs too small to fill the chip with the tiles of
// pq_qgemm.hip, or with too few steps of K to pay for their pipelines.
//
// The waves of a workgroup split K between them: wave w of KS takes the 64-wide steps w, w + KS, ... of a tile of
// 32 x 32 to 64 x 96 outputs, and the partial sums are added in a fixed order through LDS at the end.  Nothing else is
// shared: in the panel layout a fragment of 32 rows and one step is 1 KB of consecutive codes, so a wave loads its
// fragments straight into the registers the matrix unit reads, two of its steps ahead, and unpacks them there.  No
// operand goes through LDS and the loop has no barrier (row-major operands of larger outputs: see ROWS).
//
// What bounds it.  The small ones are a chain: launch, one load, the unpack and the product of a few steps, the sums.
// A 128 x 128 tile of four waves, which these shapes took before, spends 0.35 to 0.7 us in every step and
// walks all of K alone.  The larger ones are bound by the sum of matrix and vector instructions (the two overlap
// in part only, see pq_qgemm_group.hip): a 64 x 96 tile unpacks five fragments for six 32 x 32 x 64 products, 1.5 times what
// a staged 128 x 128 tile unpacks, but its four-wave workgroups need no barrier and run two to a compute unit.  Where there
// is a second workgroup, four waves and not eight share a 64 x 96 tile because it then covers the first one's ends
// (NVFP4 512 x 9216 x 3072: with eight waves 1.3 times as long); where there is none see choose_tile.  Beside a matrix
// instruction of 32 cycles seven vector instructions are free (each takes an issue slot of 4.2 cycles, the matrix
// instruction one).  So the loop tests nothing that only the last step needs (see CUT), tiles of several blocks unpack the next
// 16 k between the matrix instructions of these, in an order that is prescribed, and a wave with a single step
// runs nothing ahead.  Kernel alone, us: with 128 x 128 tiles -> split tiles -> the loop as it is and the factors in LDS
//   NVFP4     256 x 512 x 512     9.4 ->  3.6 ->  2.9     512 x 3072 x 3072   30 -> 13.4 -> 11.4     500 x 1021 x 352  3.9 -> 3.35
//   NVFP4     512 x 9216 x 3072    44 -> 32.3 -> 27.6     64 x 12288 x 3072   29 -> 10.2 ->  8.7     43 x 3659 x 10240  12.2 -> 11.2
//   INT4 g128  77 x 1000 x 1152  15.3 ->  4.3 ->  3.9     INT4 g64   1024 x 3072 x 3072  33 -> 24.9 -> 21.2
//   INT3 g64  512 x 3072 x 3072    31 -> 12.0 -> 10.2     INT3 g64   2048 x 3072 x 3072  49 -> 29.5 -> 28.7
// INT4 in the 8-bit form of pq_qgemm_group.hip gained nothing here (15.5 -> 16.5, 46.9 -> 43.6 us): fp16 operands.  For the codes
// of INT3 the next step's unpack between these blocks was 8 to 13 % slower (254 registers).
#include <type_traits>

#include "pq_qgemm_common.h"

namespace pq {

// What the matrix unit is fed with: fp16 operands that carry their group's scale (pq_qgemm.hip), or the codes with
// the scales outside (pq_qgemm_group.hip)
enum SplitMode : int { kSplitNvfp4 = 0, kSplitInt = 1, kSplitE2m1 = 2 };

// LDS bytes of the partial sums of one 32-column strip (and the flags of kWideCodes), or of two sets of steps of row-major
// operands; the epilogue's factors lie behind them
template <int TM, int TN, int KS, int WIDE, bool ROWS>
constexpr size_t split_lds();

// LDS layout of one set of KS steps of row-major operands
template <int TM, int TN, int KS>
struct RowSet {
  static constexpr int kRows = (TM + TN) * 32;
  static constexpr int kRow = KS * 32 + 16;            // bytes of a row's codes and one spare piece: the 16-byte reads of
                                                       // 32 rows at one position spread over all banks
  static constexpr int kScales = kRows * kRow;         // then two bytes a slice
  static constexpr int kScaleRow = KS * 4 + 4;
  static constexpr int kBytes = (kScales + kRows * kScaleRow + 15) / 16 * 16;
};

template <int TM, int TN, int KS, int WIDE, bool ROWS>
constexpr size_t split_lds() {
  constexpr size_t sums = (size_t)KS * TM * 32 * (32 + 4) * 4 + (WIDE == kWideCodes ? KS * 4 : 0);
  constexpr size_t sets = ROWS ? 2 * (size_t)RowSet<TM, TN, KS>::kBytes : 0;
  return sums > sets ? sums : sets;
}

typedef uint32_t uint32_any __attribute__((aligned(2)));              // two scale units, at any unit

// What int_scale_prep_kernel leaves in the workspace, for pq_qgemm_run: units and factors of block's T / 16 rows, A's and then
// W's, 16 lanes a row.  A product that prepares its scales itself has a workgroup for each block beside those of its tiles (75
// shapes 1.003 of the time without; in the first tiles' own workgroups 1.13, up to 1.28).
template <int T>
__host__ __device__ constexpr int scale_blocks(int rows) { return (rows + T / 16 - 1) / (T / 16); }
template <int T>
__device__ __forceinline__ void leave_scales(const OperandView& A, const OperandView& W, int M, int N, int groups,
                                             const RawScales& raw, int block) {
  const bool is_w = block >= scale_blocks<T>(M);
  const int row = (is_w ? block - scale_blocks<T>(M) : block) * (T / 16) + (int)threadIdx.x / 16, g0 = threadIdx.x & 15;
  if (row >= (is_w ? N : M)) return;                   // all lanes of a row; blocks past the last
  const uint8_t* scales = is_w ? W.scales + (int64_t)row * W.sc_row : A.scales + (int64_t)row * A.sc_row;
  const float* s = reinterpret_cast<const float*>(scales);
  uint16_t* units = (is_w ? raw.w_units : raw.a_units) + (int64_t)row * groups;
  float mx = 0.0f;
#pragma unroll 4
  for (int g = g0; g < groups; g += 16) mx = fmaxf(mx, int_group_max(s[g], raw.q));
  const RowScale scale = int_row_scale(group_max<16>(mx));
#pragma unroll 1
  for (int g = g0; g < groups; g += 16) units[g] = int_scale_unit(s[g], raw.q, scale.down);
  if (g0 == 0) (is_w ? raw.w_mul : raw.a_mul)[row] = scale.up / raw.q;
}

// ROWS (row-major operands only): a fragment read straight from a row-major operand touches a line for each of its 32
// rows and takes a quarter of it.  Here the workgroup loads the codes and scale units of its next KS steps together,
// whole runs of 32 KS bytes of every row, and the waves pick their step out of LDS (two sets of steps, a barrier for
// each).  The sums are the same as without, and as those of the packed operands, bit for bit.  See rows_through_lds.
// WIDE (kSplitE2m1): how codes that E2M1 does not hold are found
template <int TM, int TN, int WIDE, bool ROWS, bool FEW>
constexpr int kSplitWaves = (ROWS || WIDE == kWideMarks) && TM * TN == 4 && WIDE != kWideCodes && !FEW ? 3 : 2;      // a SIMD's; kWideCodes would spill
// FEW: at most four waves a SIMD are wanted, so that the compiler spends registers on loads further ahead (32 x 32: 84 instead
// of 58, which is two workgroups a unit instead of four; 64 x 32: 116 instead of 89, two workgroups either way).  INT3 codes, 64 x 64:
// two waves instead of three (184 registers instead of 162), and blocks in the compiler's order.
// kSplitFull: without FEW the four workgroups a unit of the 32 x 32 tiles have to be demanded (eight waves a SIMD, 64 registers; the
// compiler's own choice is 74 to 84): 72 NVFP4 shapes of more than 512 tiles and K up to 512 0.92 of the time without, 417 integer
// ones 0.99, row-major the same.
template <int MODE, int TM, int TN, int OUT, bool FEW>
constexpr bool kSplitFull = MODE != kSplitE2m1 && TM * TN == 1 && OUT != kOutDiff && !FEW;
// RAW (row-major INT operands): the scales are the quantizers' fp32 ones.  The workgroup finds its rows' largest and a lane
// turns each scale that it loads into the operand's unit.  Workgroups beside those of the tiles leave units and factors in the
// workspace.  See split_takes_raw_scales.
template <int MODE, int TM, int TN, int KS, int OUT, int WIDE, bool ROWS, bool FEW, bool RAW>
__global__ __launch_bounds__(KS * 64) __attribute__((amdgpu_waves_per_eu(kSplitFull<MODE, TM, TN, OUT, FEW> ? 8 : kSplitWaves<TM, TN, WIDE, ROWS, FEW>, FEW ? 4 : 8))) void
qgemm_split_kernel(
    OperandView A, OperandView W, int M, int N, int K, int g_shift, KernelOutput<OUT, RAW> out, int tiles_m, int tiles_n) {
  if constexpr (OUT == kOutDiff) enter_problem(A, W, out);
  constexpr int T = KS * 64;
  constexpr int BM = TM * 32, BN = TN * 32;
  constexpr bool CODES = MODE == kSplitE2m1;
  constexpr int PD = 2;                                // own steps in flight
  constexpr int ROW = 32 + 4;                          // floats of a partial sum's row in LDS
  extern __shared__ __attribute__((aligned(16))) float part[];        // [KS][BM][ROW]: one 32-column strip; then [KS] flags

  if constexpr (RAW) {                                 // told by a register: the tiles' workgroups wait for no argument here
    if (blockIdx.y) {
      leave_scales<T>(A, W, M, N, K >> g_shift, out.raw, (int)(blockIdx.y - 1) * (tiles_m * tiles_n) + (int)blockIdx.x);
      return;
    }
  }
  int tile_m, tile_n;
  assign_tile(tiles_m, tiles_n, tile_m, tile_n);
  const int tid = threadIdx.x, lane = tid & 63;
  const int ks = __builtin_amdgcn_readfirstlane(tid >> 6);            // this wave's share of K: steps ks, ks + KS, ...
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int frag_row = lane & 31, frag_half = lane >> 5;

  constexpr bool INT = MODE != kSplitNvfp4;            // factors of magnitude, the sign a mark
  const float nv_mul = INT ? 0.0f : A.mul[0] * W.mul[0];
  static_assert(!RAW || (INT && !ROWS), "fp32 scales are read directly");
  float* const factors = part + split_lds<TM, TN, KS, WIDE, ROWS>() / 4;
  Factors<BM, BN, T, INT && !RAW> own_factors;
  own_factors.load(A, W, M, N, m0, n0);

  // a fragment's lane: row lane % 32, k 32 * (lane / 32) .. + 31 of the step: 16 bytes of codes, one scale unit (packed
  // operands; see below for ROWS).  Rows past the last re-read it; what they give is not stored.
  const bool per_half = g_shift == 5;                  // a scale unit covers 32 k: the lane halves have their own
  const uint32_t half_codes = frag_half * 16u, half_a = per_half ? frag_half * (uint32_t)A.sc_step : 0u,
                 half_w = per_half ? frag_half * (uint32_t)W.sc_step : 0u;
  uint32_t a_coff[TM], w_coff[TN], a_soff[TM], w_soff[TN];
#pragma unroll
  for (int j = 0; j < TM; ++j) {
    const uint32_t r = (uint32_t)min(j * 32 + frag_row, M - 1 - m0);
    a_coff[j] = r * (uint32_t)A.code_row + half_codes;
    a_soff[j] = r * (uint32_t)A.sc_row + half_a;
  }
#pragma unroll
  for (int i = 0; i < TN; ++i) {
    const uint32_t r = (uint32_t)min(i * 32 + frag_row, N - 1 - n0);
    w_coff[i] = r * (uint32_t)W.code_row + half_codes;
    w_soff[i] = r * (uint32_t)W.sc_row + half_w;
  }
  const uint8_t* a_codes = A.codes + (int64_t)m0 * A.code_row;
  const uint8_t* w_codes = W.codes + (int64_t)n0 * W.code_row;
  const uint8_t* a_scales = A.scales + (int64_t)m0 * A.sc_row;
  const uint8_t* w_scales = W.scales + (int64_t)n0 * W.sc_row;
  const int ksteps = (K + kBK - 1) / kBK;

  struct Step {
    Slice a[TM], w[TN];
  };
  using unit_t = std::conditional_t<RAW, uint32_t, uint16_t>;
  // A step past the last re-reads the last.  CUT: K ends in a step of 32 k; its missing upper half re-reads the lower one,
  // neutralised by a zero scale.  Other K have a loop without these tests: with them the 64 x 96 tile of NVFP4 takes 8.6 vector
  // instructions for a matrix instruction, without 7.3.
  auto load = [&](auto CUT, int step, Step& f) {
    const int st = min(step, ksteps - 1);              // uniform
    const bool drop = decltype(CUT)::value && st * kBK + 32 >= K;      // uniform
    const uint32_t dc = drop ? half_codes : 0u, da = drop ? half_a : 0u, dw = drop ? half_w : 0u;
    auto at = [](uint32_t off, uint32_t less) {
      uint32_t o = off - less;
      if constexpr (!decltype(CUT)::value) asm("" : "+v"(o));           // stays 32 bits: widened ahead of the loop it takes two
      return o;                                                         // registers and a 64-bit addition a load
    };
    const int unit = (st * kBK) >> g_shift;
    const uint8_t *ac = a_codes + (int64_t)st * A.code_step, *wc = w_codes + (int64_t)st * W.code_step;
    const uint8_t *as = a_scales + (int64_t)unit * A.sc_step, *ws = w_scales + (int64_t)unit * W.sc_step;
#pragma unroll
    for (int j = 0; j < TM; ++j) {
      f.a[j].codes = *reinterpret_cast<const uint4*>(ac + at(a_coff[j], dc));
      f.a[j].sc = *reinterpret_cast<const unit_t*>(as + at(a_soff[j], da));
    }
#pragma unroll
    for (int i = 0; i < TN; ++i) {
      f.w[i].codes = *reinterpret_cast<const uint4*>(wc + at(w_coff[i], dc));
      f.w[i].sc = *reinterpret_cast<const unit_t*>(ws + at(w_soff[i], dw));
    }
  };

  float16_t acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  float a_down[RAW ? TM : 1], w_down[RAW ? TN : 1];    // of this lane's rows
  float Q = 0.0f;
  if constexpr (RAW) Q = out.raw.q;
  auto unit_of = [&](uint32_t sc, float down) -> uint32_t {
    if constexpr (RAW) return int_scale_unit(as_f32(sc), Q, down);
    else return sc;
  };
  // RAW: the factors of the tile's rows and columns to LDS, eight lanes a row, and what the scales are multiplied with here
  auto prepare_rows = [&]() {
    float* const downs = factors + kFactorBytes<BM, BN> / 4;
    const int groups = K >> g_shift;
#pragma unroll
    for (int r0 = 0; r0 < BM + BN; r0 += T / 8) {
      const int r = r0 + tid / 8, g0 = tid % 8;
      const bool mine = r < BM + BN;
      const int row = mine ? r : 0;
      const float* s = reinterpret_cast<const float*>(
          row < BM ? a_scales + (int64_t)min(row, M - 1 - m0) * A.sc_row : w_scales + (int64_t)min(row - BM, N - 1 - n0) * W.sc_row);
      float mx = 0.0f;
#pragma unroll 4
      for (int g = g0; g < groups; g += 8) mx = fmaxf(mx, int_group_max(s[g], Q));
#pragma unroll
      for (int by = 1; by < 8; by <<= 1) mx = fmaxf(mx, __shfl_xor(mx, by, kWave));
      const RowScale scale = int_row_scale(mx);
      if (mine && g0 == 0) {
        factors[r] = scale.up / Q;
        downs[r] = scale.down;
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < TM; ++j) a_down[RAW ? j : 0] = downs[j * 32 + frag_row];
#pragma unroll
    for (int i = 0; i < TN; ++i) w_down[RAW ? i : 0] = downs[BM + i * 32 + frag_row];
  };

  uint32_t wide = 0;
  // What the matrix unit takes for a share of a step: fp16 operands of 16 k (four shares), or the codes of all 64 k (one).
  constexpr int FMT = MODE == kSplitNvfp4 ? kNvfp4 : kInt4;           // INT3 nibbles unpack like INT4's
  struct Frags {
    std::conditional_t<CODES, int4v, half8_t> a[TM], w[TN];
    uint32_t sa[CODES ? TM : 1], sw[CODES ? TN : 1];
  };
  PairScale sa[CODES ? 1 : TM][2], sw[CODES ? 1 : TN][2];             // of the step that is being unpacked
  auto unpack = [&](auto KK, const Step& f, bool k_ok, Frags& to) {
    constexpr int kk = decltype(KK)::value;
    auto one = [&](const Slice& raw, PairScale (&sc)[2], float down) {
      Slice s = raw;
      if constexpr (RAW && !CODES && kk == 0) s.sc = unit_of(raw.sc, down);
      if constexpr (CODES) {
        const uint4& c = s.codes;
        if constexpr (WIDE == kWideCodes) wide |= wide_codes(c.x) | wide_codes(c.y) | wide_codes(c.z) | wide_codes(c.w);
        return (int4v){(int)e2m1_nibbles(c.x), (int)e2m1_nibbles(c.y), (int)e2m1_nibbles(c.z), (int)e2m1_nibbles(c.w)};
      } else {
        if constexpr (kk == 0) slice_scales<FMT>(s, k_ok, sc[0], sc[1]);
        const uint32_t d = kk == 0 ? s.codes.x : kk == 1 ? s.codes.y : kk == 2 ? s.codes.z : s.codes.w;
        const PairScale& h = sc[kk / 2];
        return __builtin_bit_cast(half8_t, make_uint4(unpack_pair<FMT, 0>(d, h), unpack_pair<FMT, 1>(d, h),
                                                      unpack_pair<FMT, 2>(d, h), unpack_pair<FMT, 3>(d, h)));
      }
    };
#pragma unroll
    for (int j = 0; j < TM; ++j) {
      to.a[j] = one(f.a[j], sa[CODES ? 0 : j], a_down[RAW ? j : 0]);
      if constexpr (CODES) to.sa[j] = unit_of(f.a[j].sc, a_down[RAW ? j : 0]);
    }
#pragma unroll
    for (int i = 0; i < TN; ++i) {
      to.w[i] = one(f.w[i], sw[CODES ? 0 : i], w_down[RAW ? i : 0]);
      if constexpr (CODES) to.sw[i] = frag_half == 0 ? unit_of(f.w[i].sc, w_down[RAW ? i : 0]) : 0u;
    }
  };
  auto multiply = [&](const Frags& f) {
    const float16_t zero = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f,
                            0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int j = 0; j < TM; ++j) {
        if constexpr (!CODES) {
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(f.w[i], f.a[j], acc[i][j], 0, 0, 0);
        } else {
          const int8v w = {f.w[i].x, f.w[i].y, f.w[i].z, f.w[i].w, 0, 0, 0, 0}, x = {f.a[j].x, f.a[j].y, f.a[j].z, f.a[j].w, 0, 0, 0, 0};
          const float16_t s = __builtin_amdgcn_mfma_f32_32x32x8f16(scale_operand(f.sw[i]), scale_operand(f.sa[j]), zero, 0, 0, 0);
          const float16_t p = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(w, x, zero, 4, 4, 0, 0, 0, 0);
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[i][j][r] = __builtin_fmaf(p[r], s[r], acc[i][j][r]);
          // a block at a time where three workgroups share a unit: the compiler's own order takes more than 168 registers
          if constexpr (TM * TN == 4 && !FEW) __builtin_amdgcn_sched_barrier(0);
        }
      }
  };
  auto whole_step = [&](const Step& step, bool k_ok) {
    Frags f;
    unpack(IntC<0>{}, step, k_ok, f);
    multiply(f);
    if constexpr (!CODES) {
      unpack(IntC<1>{}, step, k_ok, f);
      multiply(f);
      unpack(IntC<2>{}, step, k_ok, f);
      multiply(f);
      unpack(IntC<3>{}, step, k_ok, f);
      multiply(f);
    }
  };
  constexpr bool kAhead = !CODES && TM * TN >= 2;
  // the order of a share's instructions: the next share's unpack between this one's matrix instructions
  auto interleave = [&]() {
    if constexpr (!CODES) {
      constexpr int kUnpack = (TM + TN) * (FMT == kNvfp4 ? 8 : 11), N = TM * TN, EACH = (kUnpack + N - 1) / N;
#pragma unroll
      for (int t = 0; t < N; ++t) {
        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x2, EACH, 0);
      }
    }
  };

  if constexpr (!ROWS) {
    Step raw[PD];
    const int n_own = (ksteps - ks + KS - 1) / KS;     // steps ks, ks + KS, ...
    auto all_steps = [&](auto CUT) {
#pragma unroll
      for (int p = 0; p < PD; ++p) load(CUT, ks + p * KS, raw[p]);
      if constexpr (RAW) prepare_rows();
      auto k_ok = [&](int o) { return !decltype(CUT)::value || (ks + o * KS) * kBK + frag_half * 32 < K; };
      if constexpr (!kAhead) {
        for (int o = 0; o < n_own; o += PD) {
#pragma unroll
          for (int p = 0; p < PD; ++p) {
            if (o + p < n_own) {                       // uniform
              whole_step(raw[p], k_ok(o + p));
              load(CUT, ks + (o + p + PD) * KS, raw[p]);
            }
          }
        }
      } else {
        Frags f[2];
        unpack(IntC<0>{}, raw[0], k_ok(0), f[0]);
        for (int o = 0; o < n_own; o += PD) {
#pragma unroll
          for (int p = 0; p < PD; ++p) {
            if (o + p < n_own) {                       // uniform
              unpack(IntC<1>{}, raw[p], k_ok(o + p), f[1]);
              multiply(f[0]);
              interleave();
              unpack(IntC<2>{}, raw[p], k_ok(o + p), f[0]);
              multiply(f[1]);
              interleave();
              unpack(IntC<3>{}, raw[p], k_ok(o + p), f[1]);
              multiply(f[0]);
              interleave();
              load(CUT, ks + (o + p + PD) * KS, raw[p]);
              unpack(IntC<0>{}, raw[(p + 1) % PD], k_ok(o + p + 1), f[0]);
              multiply(f[1]);
              interleave();
              __builtin_amdgcn_sched_barrier(0);
            }
          }
        }
      }
    };
    if (ksteps <= KS) {                                // a step each at most: nothing to run ahead of
      if (RAW || ks < ksteps) load(IntC<!CODES>{}, ks, raw[0]);
      if constexpr (RAW) prepare_rows();
      if (ks < ksteps) {
        whole_step(raw[0], ks * kBK + frag_half * 32 < K);
      }
    } else if (!CODES && K % kBK)
      all_steps(IntC<!CODES>{});
    else
      all_steps(IntC<0>{});
  } else {
    // set: [rows of A, then of W] of KS steps; a row's codes with one spare piece, then the scale units of all rows: one for
    // each slice, or (CODES) a row's consecutive units of the set, of which the last set has the last ones of the row
    using L = RowSet<TM, TN, KS>;
    unsigned char* lds = reinterpret_cast<unsigned char*>(part);
    // thread t has slice t % (2 KS) of the set's 2 KS, of row t / (2 KS) of each 32
    const int slot = tid % (2 * KS), ld_row = tid / (2 * KS), ld_half = slot & 1;
    int4v codes[TM + TN];                              // the thread's slices of the set to come
    uint32_t coff[TM + TN];
#pragma unroll
    for (int q = 0; q < TM + TN; ++q) {
      const int row = q < TM ? min(q * 32 + ld_row, M - 1 - m0) : min((q - TM) * 32 + ld_row, N - 1 - n0);
      coff[q] = (uint32_t)row * (uint32_t)(q < TM ? A.code_row : W.code_row);
    }
    // CODES: KS / 2 threads share a row's units of a set, two each for groups of 64, else one.  Registers decide here: with a
    // unit for each slice the 64 x 64 tile has 174 and two workgroups on a compute unit, so 168 and three (52 shapes of more
    // than 256 tiles: 0.83 of the time).  The fp16 operands need fewer, and their units by slice are 1 to 3 % faster than this.
    constexpr int NU = CODES ? (L::kRows * (KS / 2) + T - 1) / T : TM + TN;
    const int set_units = KS * kBK >> g_shift, last_units = (K >> g_shift) - set_units;      // >= 0, see rows_through_lds
    const int piece = g_shift == 6 ? 2 : 1;
    const int sc_piece = min(tid % (KS / 2) * piece, set_units - piece) * 2, sc_row = tid / (KS / 2);
    const uint8_t* sc_from[NU];
    uint32_t soff[NU];
    std::conditional_t<CODES, uint32_t, uint16_t> units[NU];
#pragma unroll
    for (int i = 0; i < NU; ++i) {
      if constexpr (CODES) {
        const int row = sc_row + i * (T / (KS / 2));
        sc_from[i] = (row < BM ? a_scales + (int64_t)min(row, M - 1 - m0) * A.sc_row
                               : w_scales + (int64_t)min(row - BM, N - 1 - n0) * W.sc_row) + sc_piece;
      } else {
        const int row = i < TM ? min(i * 32 + ld_row, M - 1 - m0) : min((i - TM) * 32 + ld_row, N - 1 - n0);
        soff[i] = (uint32_t)row * (uint32_t)(i < TM ? A.sc_row : W.sc_row);
      }
    }
    auto fetch = [&](int set) {
      const int st = min(set * KS + (slot >> 1), ksteps - 1);
      const int half = st * kBK + ld_half * 32 < K ? ld_half : 0;
      const uint32_t k0 = (uint32_t)(st * 32 + half * 16);
      const uint32_t slice_unit = 2u * (uint32_t)(((st * kBK) >> g_shift) + (per_half ? half : 0));
#pragma unroll
      for (int q = 0; q < TM + TN; ++q) {
        codes[q] = *reinterpret_cast<const int4v*>((q < TM ? a_codes : w_codes) + (coff[q] + k0));
        if constexpr (!CODES)
          units[q] = *reinterpret_cast<const uint16_t*>((q < TM ? a_scales : w_scales) + (soff[q] + slice_unit));
      }
      if constexpr (CODES) {
        const int first = min(set * set_units, last_units) * 2;
#pragma unroll
        for (int i = 0; i < NU; ++i) {
          if (g_shift == 6)
            units[i] = *reinterpret_cast<const uint32_any*>(sc_from[i] + first);
          else
            units[i] = *reinterpret_cast<const uint16_t*>(sc_from[i] + first);
        }
      }
    };
    auto put = [&](unsigned char* set) {
#pragma unroll
      for (int q = 0; q < TM + TN; ++q) {
        const int r = q * 32 + ld_row;
        *reinterpret_cast<int4v*>(set + r * L::kRow + slot * 16) = codes[q];
        if constexpr (!CODES) *reinterpret_cast<uint16_t*>(set + L::kScales + r * L::kScaleRow + slot * 2) = units[q];
      }
      if constexpr (CODES) {
#pragma unroll
        for (int i = 0; i < NU; ++i) {
          const int row = sc_row + i * (T / (KS / 2));
          if (L::kRows * (KS / 2) % T != 0 && row >= L::kRows) continue;
          unsigned char* to = set + L::kScales + row * L::kScaleRow + sc_piece;
          if (g_shift == 6)
            *reinterpret_cast<uint32_t*>(to) = units[i];
          else
            *reinterpret_cast<uint16_t*>(to) = (uint16_t)units[i];
        }
      }
    };
    const int mine = 2 * ks + frag_half;
    const int n_sets = (ksteps + KS - 1) / KS;
    // set o: out of LDS stage o % 2, while set o + 1 goes into the other one, which was last read before the barrier
    // in between, and set o + 2 is asked for
    auto turn = [&](auto Pc, int o) {
      constexpr int P = decltype(Pc)::value;           // o % 2
      const unsigned char* have = lds + P * L::kBytes;
      const int step = o * KS + ks;
      const int unit = CODES ? (min(step, ksteps - 1) * kBK >> g_shift) - min(o * set_units, last_units) : mine;
      const unsigned char* have_sc = have + L::kScales + unit * 2;
      Step own;
#pragma unroll
      for (int q = 0; q < TM; ++q) {
        own.a[q].codes = *reinterpret_cast<const uint4*>(have + (q * 32 + frag_row) * L::kRow + mine * 16);
        own.a[q].sc = *reinterpret_cast<const uint16_t*>(have_sc + (q * 32 + frag_row) * L::kScaleRow);
      }
#pragma unroll
      for (int q = 0; q < TN; ++q) {
        own.w[q].codes = *reinterpret_cast<const uint4*>(have + ((TM + q) * 32 + frag_row) * L::kRow + mine * 16);
        own.w[q].sc = *reinterpret_cast<const uint16_t*>(have_sc + ((TM + q) * 32 + frag_row) * L::kScaleRow);
      }
      if (o + 1 < n_sets) {                            // uniform over the workgroup
        put(lds + (P ^ 1) * L::kBytes);
        fetch(o + 2);
      }
      if (step < ksteps) {                             // uniform over the wave
        whole_step(own, step * kBK + frag_half * 32 < K);
      }
      __syncthreads();
    };
    fetch(0);
    put(lds);
    own_factors.put(factors);                            // here, where the loads are waited for anyway
    fetch(1);
    __syncthreads();
    for (int o = 0; o < n_sets; o += 2) {
      turn(IntC<0>{}, o);
      if (o + 1 < n_sets) turn(IntC<1>{}, o + 1);      // uniform over the workgroup
    }
  }

  if constexpr (!RAW && !ROWS) own_factors.put(factors);

  // ---- the partial sums meet in LDS, one 32-column strip at a time, and are added in a fixed order
  const bool bias = !RAW && W.bias != nullptr;         // RAW: refused at the launch, nothing puts it into LDS
  void* __restrict__ y = out.y;
  const int64_t ldy = out.ldy;
  double d2 = 0.0;
  constexpr int CHUNKS = 4;                            // eight columns each
  constexpr float unit = CODES ? 4.0f : 1.0f;          // undoes the E2M1 codes' factor 1/2 on either side
#pragma unroll
  for (int i = 0; i < TN; ++i) {
    if (i) __syncthreads();
#pragma unroll
    for (int j = 0; j < TM; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float* p = part + (size_t)(ks * BM + j * 32 + frag_row) * ROW + q * 8 + frag_half * 4;
        *reinterpret_cast<float4*>(p) =
            make_float4(acc[i][j][q * 4], acc[i][j][q * 4 + 1], acc[i][j][q * 4 + 2], acc[i][j][q * 4 + 3]);
      }
    __syncthreads();
    for (int c = tid; c < BM * CHUNKS; c += T) {
      const int row = c / CHUNKS, cc = c % CHUNKS;
      const int m = m0 + row, n = n0 + i * 32 + cc * 8;
      if (m >= M || n >= N) continue;
      float v[8];
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const float4* p = reinterpret_cast<const float4*>(part + (size_t)(s * BM + row) * ROW + cc * 8);
        const float4 lo = p[0], hi = p[1];
        const float t[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = s == 0 ? t[e] : v[e] + t[e];
      }
      const float* col = factors + BM + i * 32 + cc * 8;
      if constexpr (INT) {
        const float am = fabsf(factors[row]);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = (v[e] * unit) * (am * fabsf(col[e]));
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] *= nv_mul;
      }
      if (bias) {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += col[BN + e];
      }
      if constexpr (OUT == kOutDiff) {
        const float* r = out.ref + (int64_t)m * ldy + n;
        float f[8];
        if (n + 7 < N) {
          const float4 lo = *reinterpret_cast<const float4*>(r), hi = *reinterpret_cast<const float4*>(r + 4);
          f[0] = lo.x; f[1] = lo.y; f[2] = lo.z; f[3] = lo.w;
          f[4] = hi.x; f[5] = hi.y; f[6] = hi.z; f[7] = hi.w;
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            f[e] = n + e < N ? r[e] : 0.0f;
            v[e] = n + e < N ? v[e] : 0.0f;            // no column: no difference
          }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const double d = (double)f[e] - (double)v[e];
          d2 = fma(d, d, d2);
        }
      } else if constexpr (OUT == kOutF32) {
        float* yo = reinterpret_cast<float*>(y) + (int64_t)m * ldy + n;
        if (n + 7 < N) {
          *reinterpret_cast<float4*>(yo) = make_float4(v[0], v[1], v[2], v[3]);
          *reinterpret_cast<float4*>(yo + 4) = make_float4(v[4], v[5], v[6], v[7]);
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (n + e < N) yo[e] = v[e];
        }
      } else {
        uint16_t* yo = reinterpret_cast<uint16_t*>(y) + (int64_t)m * ldy + n;
        uint32_t w[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = cvt_pk_bf16(v[2 * e], v[2 * e + 1]);
        if (n + 7 < N) {
          *reinterpret_cast<uint4*>(yo) = make_uint4(w[0], w[1], w[2], w[3]);
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (n + e < N) yo[e] = (uint16_t)(w[e >> 1] >> (16 * (e & 1)));
        }
      }
    }
  }
  if constexpr (OUT == kOutDiff) {
    __syncthreads();                                   // the partial sums have been read
    store_diff(d2, reinterpret_cast<double*>(part), T, tile_m * tiles_n + tile_n, out);
  }
  if constexpr (WIDE != kWideNone) {                   // here, where the accumulators are dead
    const bool any = WIDE == kWideMarks ? __any((int)tile_marks<BM, BN>(factors) < 0) != 0
                                        : any_wide<KS>(wide, reinterpret_cast<int*>(part + (size_t)KS * BM * ROW));
    if (any) {
      __threadfence();                                 // what the waves stored has arrived
      __syncthreads();
      wide_codes_tile<BM, BN, KS, KS, OUT, RAW>(A, W, M, N, K, g_shift, m0, n0, out, factors);
    }
  }
}

// Whether a product of row-major operands reads them through LDS (tiles of 64 rows with eight waves always do, see
// split_eight).  Up to one workgroup a unit its chain of loads is what
// takes the time, and the direct loads are two steps ahead without a barrier (INT4 g128 77 x 1000 x 1152, 96 tiles: 7.0 us
// direct, 7.8 through LDS; 212 shapes 0.71 to 1.20).  With more, the lines of a unit's workgroups push each other out of its
// cache before all of their quarters are read.  A first set has to be full, and a few steps have to pay for the barriers.
// Measured over 433 shapes of more than 256 tiles, at the tiles that they take, through LDS against direct: tiles of eight
// waves from a full set on 0.55 to 1.03; of four waves from 4 steps on where every row starts at a line (K a multiple of
// 256) 0.46 to 0.99, else from 6 steps on 0.56 to 1.05 (before that 0.97 to 1.06).  us, direct | through LDS | the staged
// tiles that these shapes took once: NVFP4 2048 x 3072 x 3072 73 | 48 | 56, 512 x 9216 x 3072 57 | 37 | 53, INT4 g64
// 1024 x 3072 x 3072 41 | 32 | 38, INT3 g64 2048 x 3072 x 3072 84 | 41 | 59.
static bool rows_through_lds(int64_t n_tiles, int ks, int K) {
  return n_tiles > 256 && K >= (ks == 8 ? 8 : K % 256 == 0 ? 4 : 6) * kBK;
}

// Whether a product of row-major INT operands prepares their scales itself (RAW) instead of in a launch before it, which
// takes 1.3 to 2.5 us of the device and 2.7 of the host, and as long as it takes to read all codes where it looks for INT3 codes beyond
// three bits.  Every workgroup then reads all scales of its rows ahead of its first step and loads two bytes more a unit.  With
// many groups a row that is longer than the launch, with a long K where every row starts at a line of the cache (K a multiple of
// 256) because the rows' lines push each other out, and earlier where a workgroup has 64 rows.  Random shapes of at most 256
// tiles (1 to 2048 rows, 64 to 8192 columns, K 96 to 12288, all groups), device alone: the lines were drawn on 5400 and take 4687 of them in
// 0.77 of the time of the launch and the product, two more than 1.01 and at most 1.045; of 6000 others, all with K from 1800 on, 3947 in
// 0.85, 18 more than 1.01, at most 1.052.  Beyond the lines 0.96, up to 1.20 (INT3 g64 1009 x 502 x 3584 15.5 -> 18.5 us, INT4 g256 768 x 384 x
// 6144 20.3 -> 23.4).  us: INT4 g128 77 x 1000 x 1152 6.4 -> 5.2, INT3 g128 24 x 6133 x 11904 28.2 -> 20.0.
bool split_takes_raw_scales(pq_format fmt, int group, int tile, int64_t M, int64_t N, int64_t K) {
  if (fmt == PQ_FMT_NVFP4 || (tile != kTileSplit32 && tile != kTileSplit64x32) || qgemm_tiles(tile, M, N) > 256) return false;
  const bool marks = fmt == PQ_FMT_INT3 && group != 32, lines = K % 256 == 0;
  if (marks && (M + N) * K >= 30000000) return true;
  if (tile == kTileSplit32) return K <= 5120 || (!lines && K / group <= 128);
  return K <= 2304 || (!lines && (marks || K <= 3072));
}

template <int MODE, int TM, int TN, int KS, int OUT, int WIDE, bool ROWS, bool FEW = false, bool RAW = false>
static int launch_split(const OperandView& A, const OperandView& W, int M, int N, int K, int g_shift,
                        const std::conditional_t<RAW, RawOutput, Outputs>& out, hipStream_t st) {
  constexpr int BM = TM * 32, BN = TN * 32;
  constexpr size_t shmem = split_lds<TM, TN, KS, WIDE, ROWS>() + kFactorBytes<BM, BN> + (RAW ? (BM + BN) * 4 : 0);
  static_assert(shmem <= 160 * 1024, "the partial sums fit in LDS");
  auto kern = qgemm_split_kernel<MODE, TM, TN, KS, OUT, WIDE, ROWS, FEW, RAW>;
  static std::atomic<uint64_t> raised{0};
  if (int rc = allow_lds(reinterpret_cast<const void*>(kern), shmem, raised, "hipFuncSetAttribute(qgemm_split_kernel)")) return rc;
  const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  const int64_t n_tiles = (int64_t)tiles_m * tiles_n;
  if (n_tiles > 0x7FFFFFFF) return fail(PQ_ERR_SHAPE, "too many output tiles");
  dim3 grid((unsigned)n_tiles);
  if constexpr (RAW) grid.y = (unsigned)(1 + (scale_blocks<KS * 64>(M) + scale_blocks<KS * 64>(N) + n_tiles - 1) / n_tiles);
  else grid.y = out.problems;
  hipLaunchKernelGGL(kern, grid, dim3(KS * 64), shmem, st, A, W, M, N, K, g_shift, out, tiles_m, tiles_n);
  return check_hip(hipGetLastError(), "qgemm_split_kernel");
}

// The loader of the operands' layout and the shape.  FEW as long as two workgroups a unit hold the launch: NVFP4 109 x 140 x
// 4928 (20 tiles) 12.7 us, FEW 12.2, 43 x 3659 x 10240 (230) 20.9, 19.9, 134 x 10981 x 320 (1720) 8.6, 11.2.  12500 shapes of these
// tiles against FEW throughout 0.997 (0.81 to 0.95 beyond 512 tiles), 13300 against none 0.991.  INT3 codes on 64 x 64 up to 512 tiles,
// 1740 shapes: 0.97 of the time of three workgroups a unit, K beyond 4096 0.91 (1.07 of what it was before there were three; 0.96
// with FEW); up to 700 tiles three and two take the same, beyond them three win.
template <int MODE, int TM, int TN, int KS, int OUT, int WIDE>
static int split_loader(const OperandView& A, const OperandView& W, int M, int N, int K, int g_shift, const Outputs& out,
                        hipStream_t st) {
  const int64_t n_tiles = (int64_t)((M + TM * 32 - 1) / (TM * 32)) * ((N + TN * 32 - 1) / (TN * 32));
  if constexpr (OUT != kOutDiff) {                     // the selection, which keeps the difference, packs its operands
    if (!(A.panel && W.panel) && rows_through_lds(n_tiles, KS, K))
      return launch_split<MODE, TM, TN, KS, OUT, WIDE, true>(A, W, M, N, K, g_shift, out, st);
  }
  constexpr bool kMayBeFew = MODE == kSplitE2m1 ? WIDE == kWideMarks && TM * TN == 4 : TN == 1, kFew = kMayBeFew && TM * TN == 2;
  if constexpr (kMayBeFew && !kFew) {
    if (n_tiles * out.problems <= 512)
      return launch_split<MODE, TM, TN, KS, OUT, WIDE, false, true>(A, W, M, N, K, g_shift, out, st);
  }
  return launch_split<MODE, TM, TN, KS, OUT, WIDE, false, kFew>(A, W, M, N, K, g_shift, out, st);
}

// eight waves on 64 rows (choose_tile): row-major operands go through LDS.  The direct loads of eight waves push each other's
// lines out of the cache: NVFP4 512 x 1650 x 3072 four waves 16.4 us, eight 18.6, eight through LDS 12.4.
template <int MODE, int TN, int OUT, int WIDE>
static int split_eight(const OperandView& A, const OperandView& W, int M, int N, int K, int g_shift, const Outputs& out,
                       hipStream_t st) {
  if constexpr (OUT != kOutDiff) {
    if (!(A.panel && W.panel)) return launch_split<MODE, 2, TN, 8, OUT, WIDE, true>(A, W, M, N, K, g_shift, out, st);
  }
  return launch_split<MODE, 2, TN, 8, OUT, WIDE, false, MODE == kSplitE2m1 && WIDE == kWideMarks && TN == 2>(A, W, M, N, K, g_shift, out, st);
}

template <int MODE, int OUT, int WIDE>
static int split_tile(const OperandView& A, const OperandView& W, int M, int N, int K, int g_shift, const Outputs& out,
                      int tile, hipStream_t st) {
  switch (tile) {
    case kTileSplit32: return split_loader<MODE, 1, 1, 8, OUT, WIDE>(A, W, M, N, K, g_shift, out, st);
    case kTileSplit64x32: return split_loader<MODE, 2, 1, 8, OUT, WIDE>(A, W, M, N, K, g_shift, out, st);
    case kTileSplit64: return split_loader<MODE, 2, 2, 4, OUT, WIDE>(A, W, M, N, K, g_shift, out, st);
    case kTileSplit64Eight: return split_eight<MODE, 2, OUT, WIDE>(A, W, M, N, K, g_shift, out, st);
    case kTileSplit64x96Eight: return split_eight<MODE, 3, OUT, WIDE>(A, W, M, N, K, g_shift, out, st);
    default: return split_loader<MODE, 2, 3, 4, OUT, WIDE>(A, W, M, N, K, g_shift, out, st);
  }
}

static int group_shift(pq_format fmt, int group) {
  return fmt == PQ_FMT_NVFP4 || group == 32 ? 5 : group == 64 ? 6 : group == 128 ? 7 : 8;
}

int launch_qgemm_split(pq_format fmt, int group, const OperandView& A, const OperandView& W, int M, int N, int K,
                       const Outputs& out, int tile, hipStream_t st) {
  const int g_shift = group_shift(fmt, group);
#define PQ_SPLIT(MODE, WIDE)                                                                                 \
  return out.kind == kOutF32    ? split_tile<MODE, kOutF32, WIDE>(A, W, M, N, K, g_shift, out, tile, st)      \
         : out.kind == kOutDiff ? split_tile<MODE, kOutDiff, kWideNone>(A, W, M, N, K, g_shift, out, tile, st) \
                                : split_tile<MODE, kOutBf16, WIDE>(A, W, M, N, K, g_shift, out, tile, st)
  if (fmt == PQ_FMT_NVFP4) PQ_SPLIT(kSplitNvfp4, kWideNone);
  if (fmt == PQ_FMT_INT3 && group != 32) {
    if (A.marked && W.marked) PQ_SPLIT(kSplitE2m1, kWideMarks);
    PQ_SPLIT(kSplitE2m1, kWideCodes);
  }
  PQ_SPLIT(kSplitInt, kWideNone);
#undef PQ_SPLIT
}

// Views with fp32 scales come here and nowhere else: the other kernels would read them as units, and factors where there are
// none.
template <int MODE, int OUT, int WIDE>
static int split_raw(const OperandView& A, const OperandView& W, int M, int N, int K, int g_shift, const RawOutput& out, int tile,
                     hipStream_t st) {
  constexpr bool kFew = MODE != kSplitE2m1;
  if (tile == kTileSplit32) return launch_split<MODE, 1, 1, 8, OUT, WIDE, false, kFew, true>(A, W, M, N, K, g_shift, out, st);
  return launch_split<MODE, 2, 1, 8, OUT, WIDE, false, kFew, true>(A, W, M, N, K, g_shift, out, st);
}

int launch_qgemm_split_raw(pq_format fmt, int group, const OperandView& A, const OperandView& W, int M, int N, int K,
                           const RawOutput& out, int tile, hipStream_t st) {
  if (out.kind == kOutDiff || W.bias || !split_takes_raw_scales(fmt, group, tile, M, N, K))
    return fail(PQ_ERR_FORMAT, "no product with fp32 group scales of this kind");
  const int g_shift = group_shift(fmt, group);
#define PQ_RAW(MODE, WIDE)                                                                            \
  return out.kind == kOutF32 ? split_raw<MODE, kOutF32, WIDE>(A, W, M, N, K, g_shift, out, tile, st) \
                             : split_raw<MODE, kOutBf16, WIDE>(A, W, M, N, K, g_shift, out, tile, st)
  if (fmt == PQ_FMT_INT3 && group != 32) PQ_RAW(kSplitE2m1, kWideCodes);
  PQ_RAW(kSplitInt, kWideNone);
#undef PQ_RAW
}

}  // namespace pq
