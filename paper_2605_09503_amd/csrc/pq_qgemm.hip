// Low-bit GEMM of the reordered quantized layer (paper Eq. 8):
//     Y[m, n] = Ta Tw sum_g sa[m, g] sw[n, g] sum_{k in g} a[m, k] w[n, k]
//
// Design for gfx950.  Large outputs are computed here, those of the integer formats with groups of 64 and more in
// pq_qgemm_group.hip, small outputs in pq_qgemm_split.hip; choose_tile (pq_qgemm_tile.hip) says which.
// The contraction runs on the fp16 MFMA (v_mfma_f32_32x32x16_f16, fp32
// accumulate).  Both operands stay 4-bit in HBM and L2; a workgroup unpacks its A and W tiles
// once per K step straight into fp16 values that already carry the per-group scale, and stages
// them in LDS:
//   NVFP4  value = E2M1 code * E4M3 block scale: 2 + 4 significant bits and an exponent range
//          of [2^-10, 2688] -- exact in fp16.  The two fp32 tensor scales go to the epilogue.
//   INT    the stored scale is s = fl32(h / Q) with h the group's bf16 maximum, so h is
//          recovered exactly as bf16_rne(s * Q) and the operand is z * h * 2^-E(row): 3 + 8
//          significant bits, exact in fp16; E(row) keeps the row's largest group below the
//          fp16 maximum.  2^E(row) / Q goes to the epilogue.
// The MFMA then forms exact products of the scaled operands and adds them in fp32, i.e. the
// per-group scale products are applied inside the K accumulation without any per-group pass
// over the accumulators on the vector ALU (that pass would cost 2 lane-ops per output per
// group and would bound the kernel well below the matrix pipe).
//
// Tiling: BM x BN output tile per workgroup, BK = 64 per step, double-buffered LDS, one
// barrier per step.  Waves form a WGM x WGN grid; each owns (BM/WGM) x (BN/WGN) outputs as
// 32x32 MFMA tiles.  The MFMA "A" operand is the weight tile and "B" the activation tile, so
// a lane ends up with 4 consecutive n for one m and stores 8 bytes of bf16 at once.
// LDS rows are 64 fp16 plus one 16-byte piece of padding (144 bytes): measured on gfx950, the
// 16-byte fragment reads of the 32-row MFMA operand pattern run at full LDS rate with this
// stride (an XOR swizzle of unpadded rows reaches two thirds of it).
#include <string.h>

#include "pq_qgemm_common.h"

namespace pq {

// Software pipeline of one K step s (P = s & 1 is the LDS stage being multiplied):
//   - global loads for step s + 3 are issued first (two steps ahead of their use),
//   - the MFMAs of step s run on stage P, fragment reads for the next 16-wide k slice are
//     issued one slice ahead,
//   - between MFMAs the wave unpacks its slice of step s + 1 (already in registers) pair by
//     pair and writes it to stage P ^ 1,
//   - one barrier, before the last k slice: the first fragments of step s + 1 are read during that slice.
// Every MFMA is followed by its share of vector-ALU and LDS work in program order, pinned
// with scheduling barriers, so that the matrix pipe and the vector ALU overlap inside a wave
// instead of alternating in phases.
template <int FMT, int G, int BM, int BN, int WGM, int WGN, int OUT>
__global__ __launch_bounds__(WGM* WGN * 64) void qgemm_kernel(OperandView A, OperandView W, int M, int N,
                                                              int K, KernelOutput<OUT> out,
                                                              int tiles_m, int tiles_n) {
  if constexpr (OUT == kOutDiff) enter_problem(A, W, out);
  // NVFP4: the tensor scales, in scalar registers from here on
  const float nv_mul = FMT == kNvfp4 ? A.mul[0] * W.mul[0] : 0.0f;
  constexpr int T = WGM * WGN * 64;
  // wave tile: WTM x WTN outputs.  BM need not divide evenly over the WGM wave rows: the last wave row
  // then owns TM_LAST < TM MFMA tiles along M (a 224-row tile is 128 + 96), and the waves are numbered so
  // that every SIMD hosts one wave of each kind (see below)
  constexpr int WTM = (BM + WGM * 32 - 1) / (WGM * 32) * 32, WTN = BN / WGN;
  constexpr int TM = WTM / 32, TN = WTN / 32;        // MFMA tiles per wave
  constexpr int TM_LAST = (BM - (WGM - 1) * WTM) / 32;
  constexpr bool RAGGED_M = TM_LAST != TM;
  constexpr int SL = BN * 2 / T;                     // slices per operand per thread
  static_assert(BN * 2 % T == 0 && (BM * 2 + T - 1) / T == SL, "whole slices per thread, as many for A as for W");
  static_assert(BM % 32 == 0 && WTN % 32 == 0 && TM_LAST >= 1 && TM_LAST <= TM, "wave tile");
  static_assert(!RAGGED_M || (WGM == 2 && WGN == 4), "the uneven split is laid out for 2 x 4 waves");
  // the loader covers SL * T / 2 rows of each operand; an A tile of fewer rows (BM = 224) still gets all
  // of them in LDS, so that no thread needs a predicate around its unpack writes (the spare rows hold the
  // matrix rows behind the tile and are never read)
  constexpr int A_TILE_BYTES = SL * (T / 2) * kRowBytes, W_TILE_BYTES = BN * kRowBytes;
  constexpr int STAGE_BYTES = A_TILE_BYTES + W_TILE_BYTES;

  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

  int tile_m, tile_n;
  assign_tile(tiles_m, tiles_n, tile_m, tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * BN;

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  // Waves of a workgroup go to the four SIMDs in turn (wave w on SIMD w % 4).  With the uneven split
  // waves w and w + 4 take different wave rows, so that every SIMD's matrix pipe gets TM + TM_LAST tile
  // rows of work per step.
  const int wave_m = RAGGED_M ? ((wave >> 2) ^ wave) & 1 : wave % WGM;
  const int wave_n = RAGGED_M ? wave >> 1 : wave / WGM;
  // MFMA tile rows this wave owns (wave-uniform, kept in a scalar register)
  const int tm_cnt = RAGGED_M ? __builtin_amdgcn_readfirstlane(wave_m == WGM - 1 ? TM_LAST : TM) : TM;

  // loader: this thread owns tile rows tid / 2 + q * (T / 2), k offset 32 * (tid & 1), of both
  // operands
  const int ld_row = tid >> 1, ld_half = tid & 1;
  // addresses: a uniform part (the tile, the step) and a 32-bit offset inside the tile.  Rows past the last re-read it: what
  // they give is not stored.
  uint32_t a_coff[SL], w_coff[SL], a_soff[SL], w_soff[SL];
  const uint32_t half_codes = ld_half * 16u;
  const uint32_t half_a = ld_half * (uint32_t)A.sc_step, half_w = ld_half * (uint32_t)W.sc_step;
  constexpr bool kHalfUnits = FMT == kNvfp4 || G == 32;              // a scale unit covers 32 k
#pragma unroll
  for (int q = 0; q < SL; ++q) {
    const int r = ld_row + q * (T / 2);
    const uint32_t a_row = (uint32_t)min(r, M - 1 - m0), w_row = (uint32_t)min(r, N - 1 - n0);
    a_coff[q] = a_row * (uint32_t)A.code_row + half_codes;
    w_coff[q] = w_row * (uint32_t)W.code_row + half_codes;
    a_soff[q] = a_row * (uint32_t)A.sc_row + (kHalfUnits ? half_a : 0u);
    w_soff[q] = w_row * (uint32_t)W.sc_row + (kHalfUnits ? half_w : 0u);
  }
  const uint8_t* a_codes = A.codes + (int64_t)m0 * A.code_row;
  const uint8_t* w_codes = W.codes + (int64_t)n0 * W.code_row;
  const uint8_t* a_scales = A.scales + (int64_t)m0 * A.sc_row;
  const uint8_t* w_scales = W.scales + (int64_t)n0 * W.sc_row;
  const int ksteps = (K + kBK - 1) / kBK;
  // Loads never leave the operand and never branch (a branch in the loop would split its schedule): a step past the last
  // re-reads the last, the missing upper half of a last step of 32 k the lower one.  What such a slice holds does not
  // matter: its scale is taken as zero.  (With a 64-bit address a load, a branch around what lies past the end and a mask for
  // rows past the last 2.9 vector instructions stood beside a matrix instruction, now 2.5: NVFP4 4608 x 9216 x 3072 205.1 -> 200.0
  // us, 4608 x 3072 x 12288 260.5 -> 256.4, INT3 g32 8192 x 12288 x 3072 468.9 -> 462.6.)
  auto load_ops = [&](const uint8_t* codes, const uint32_t (&coff)[SL], int code_step, const uint8_t* scales,
                      const uint32_t (&soff)[SL], int sc_step, uint32_t half_sc, int step, Slice (&r)[SL]) {
    const int st = min(step, ksteps - 1);                             // uniform
    const bool drop = st * kBK + 32 >= K;                             // uniform
    const uint32_t dc = drop ? half_codes : 0u, ds = drop && kHalfUnits ? half_sc : 0u;
    const uint8_t* c = codes + (int64_t)st * code_step;
    const uint8_t* sc = scales + (int64_t)(kHalfUnits ? 2 * st : st * kBK / G) * sc_step;
#pragma unroll
    for (int q = 0; q < SL; ++q) {
      r[q].codes = *reinterpret_cast<const uint4*>(c + (coff[q] - dc));
      r[q].sc = *reinterpret_cast<const uint16_t*>(sc + (soff[q] - ds));
    }
  };
  auto load_a = [&](int step, Slice (&ra)[SL]) { load_ops(a_codes, a_coff, A.code_step, a_scales, a_soff, A.sc_step, half_a, step, ra); };
  auto load_w = [&](int step, Slice (&rw)[SL]) { load_ops(w_codes, w_coff, W.code_step, w_scales, w_soff, W.sc_step, half_w, step, rw); };
  // byte offsets of this thread's 16-byte pieces inside an operand tile: [slot][piece]
  int st_off[SL][4];
#pragma unroll
  for (int q = 0; q < SL; ++q)
#pragma unroll
    for (int c = 0; c < 4; ++c) st_off[q][c] = lds_off(ld_row + q * (T / 2), ld_half * 4 + c);

  const int frag_row = lane & 31, frag_half = lane >> 5;
  // fragment read offsets: row part + swizzled piece for each of the four k slices
  int w_frag_base[TN], x_frag_base[TM];
#pragma unroll
  for (int i = 0; i < TN; ++i) w_frag_base[i] = (wave_n * WTN + i * 32 + frag_row) * kRowBytes;
#pragma unroll
  for (int j = 0; j < TM; ++j) x_frag_base[j] = (wave_m * WTM + j * 32 + frag_row) * kRowBytes;
  int piece_off[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) piece_off[kk] = (kk * 2 + frag_half) << 4;

  float16_t acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  Slice raw_a[2][SL], raw_w[2][SL];

  // one operand slice -> its four 16-byte pieces in LDS (used by the prologue only)
  auto unpack_all = [&](const Slice& sl, bool ok, unsigned char* tile, int q) {
    PairScale s0, s1;
    slice_scales<FMT>(sl, ok, s0, s1);
    const uint32_t d[4] = {sl.codes.x, sl.codes.y, sl.codes.z, sl.codes.w};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const PairScale& sc = c < 2 ? s0 : s1;
      uint4 v = make_uint4(unpack_pair<FMT, 0>(d[c], sc), unpack_pair<FMT, 1>(d[c], sc),
                           unpack_pair<FMT, 2>(d[c], sc), unpack_pair<FMT, 3>(d[c], sc));
      *reinterpret_cast<uint4*>(tile + st_off[q][c]) = v;
    }
  };

  // ---- prologue: stage 0 <- step 0, raw[1] <- step 1, raw[0] <- step 2
  load_a(0, raw_a[0]);
  load_w(0, raw_w[0]);
  load_a(1, raw_a[1]);
  load_w(1, raw_w[1]);
  float* const factors = reinterpret_cast<float*>(smem + 2 * STAGE_BYTES);
  {
    Factors<BM, BN, T, FMT != kNvfp4> f;
    f.load(A, W, M, N, m0, n0);
    f.put(factors);
  }
#pragma unroll
  for (int q = 0; q < SL; ++q) {
    unpack_all(raw_a[0][q], ld_half * 32 < K, smem, q);
    unpack_all(raw_w[0][q], ld_half * 32 < K, smem + A_TILE_BYTES, q);
  }
  load_a(2, raw_a[0]);
  load_w(2, raw_w[0]);
  __syncthreads();

  // weight fragments: one set, each reloaded for the next k slice right after its last MFMA; activation
  // fragments: two sets (they are used by every MFMA of a slice)
  half8_t wf[TN], xf[2][TM];
  auto read_w = [&](const unsigned char* stage, int kk, int i) {
    wf[i] = *reinterpret_cast<const half8_t*>(stage + A_TILE_BYTES + w_frag_base[i] + piece_off[kk]);
  };
  auto read_x = [&](const unsigned char* stage, int set, int kk, int j) {
    xf[set][j] = *reinterpret_cast<const half8_t*>(stage + x_frag_base[j] + piece_off[kk]);
  };
#pragma unroll
  for (int j = 0; j < TM; ++j)
    if (!RAGGED_M || j < tm_cnt) read_x(smem, 0, 0, j);
#pragma unroll
  for (int i = 0; i < TN; ++i) read_w(smem, 0, i);

  // TMc: the MFMA tile rows of the calling wave as a compile-time constant (TM, or TM_LAST for the
  // short wave row of an uneven split) -- each kind of wave runs its own straight-line loop
  auto body = [&](auto Pc, auto TMc, int s) {
    constexpr int P = decltype(Pc)::value;
    constexpr int TMW = decltype(TMc)::value;
    constexpr int NM = TN * TMW;                     // MFMAs per 16-wide k slice
    const unsigned char* stage = smem + P * STAGE_BYTES;
    const unsigned char* next = smem + (P ^ 1) * STAGE_BYTES;
    unsigned char* a_nx = smem + (P ^ 1) * STAGE_BYTES;
    unsigned char* w_nx = a_nx + A_TILE_BYTES;

    // step s + 1 sits in raw[P ^ 1]; it is unpacked during this step and the registers are
    // refilled with step s + 3 as soon as they are free
    Slice(&ca)[SL] = raw_a[P ^ 1];
    Slice(&cw)[SL] = raw_w[P ^ 1];
    PairScale sc_a[SL][2], sc_w[SL][2];
#pragma unroll
    for (int q = 0; q < SL; ++q) {
      const bool k_ok = (s + 1) * kBK + ld_half * 32 < K;
      slice_scales<FMT>(ca[q], k_ok, sc_a[q][0], sc_a[q][1]);
      slice_scales<FMT>(cw[q], k_ok, sc_w[q][0], sc_w[q][1]);
    }

    uint32_t pk[4];        // the unit (one dword of codes -> one 16-byte piece) being assembled
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const int cur = kk & 1;
      // The step's barrier stands before its last slice, whose fragments are in registers by then: the first
      // fragments of the next step are on their way while that slice is multiplied, and no wave starts a step waiting
      // for LDS.
      if (kk == 3) {
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int mi = 0; mi < NM; ++mi) {
        const int i = mi / TMW, j = mi % TMW;
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(wf[i], xf[cur][j], acc[i][j], 0, 0, 0);
        if (kk < 3) {
          if (j == TMW - 1) read_w(stage, kk + 1, i);                // wf[i] is free now
          if (mi < TMW) read_x(stage, cur ^ 1, kk + 1, mi);          // next slice's activations, early
        } else {
          if (j == TMW - 1) read_w(next, 0, i);
          if (mi < TMW) read_x(next, 0, 0, mi);
        }
        // unpack tasks: 32 SL pairs, spread evenly over the MFMAs of the first three slices (their pieces have to be in
        // LDS at the barrier).  Task order: A slot 0 (4 pieces x 4 pairs), A slot 1, ..., then the W slots.
        if (kk < 3) {
          const int slot = kk * NM + mi;             // tasks that start in it: g 3 NM / (32 SL) == slot
#pragma unroll
          for (int g = (slot * 32 * SL + 3 * NM - 1) / (3 * NM); g < ((slot + 1) * 32 * SL + 3 * NM - 1) / (3 * NM); ++g) {
            const int u = g / 4;                // unit: one dword of codes -> one LDS piece
            const int jp = g % 4;
            const bool is_w = u >= 4 * SL;
            const int q = (u / 4) % SL, c = u % 4;
            const Slice& src = is_w ? cw[q] : ca[q];
            const uint32_t d = c == 0 ? src.codes.x : c == 1 ? src.codes.y : c == 2 ? src.codes.z : src.codes.w;
            const PairScale& sc = is_w ? sc_w[q][c / 2] : sc_a[q][c / 2];
            if (jp == 0) pk[0] = unpack_pair<FMT, 0>(d, sc);
            if (jp == 1) pk[1] = unpack_pair<FMT, 1>(d, sc);
            if (jp == 2) pk[2] = unpack_pair<FMT, 2>(d, sc);
            if (jp == 3) {
              pk[3] = unpack_pair<FMT, 3>(d, sc);
              unsigned char* dst = (is_w ? w_nx : a_nx) + st_off[q][c];
              *reinterpret_cast<uint4*>(dst) = make_uint4(pk[0], pk[1], pk[2], pk[3]);
            }
            if (g == 16 * SL - 1) load_a(s + 3, ca);
            if (g == 32 * SL - 1) load_w(s + 3, cw);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };

  // two steps per trip so that the LDS stage and the register set are compile-time constants;
  // an odd step count runs one extra step, the last one's codes under scales of zero,
  // which keeps a single loop exit (two exits would double the live accumulators)
  if (!RAGGED_M || tm_cnt == TM) {
    for (int s = 0; s < ksteps; s += 2) {
      body(IntC<0>{}, IntC<TM>{}, s);
      body(IntC<1>{}, IntC<TM>{}, s + 1);
    }
  } else {
    // same number of barriers as the other kind of wave: one per step
    for (int s = 0; s < ksteps; s += 2) {
      body(IntC<0>{}, IntC<TM_LAST>{}, s);
      body(IntC<1>{}, IntC<TM_LAST>{}, s + 1);
    }
  }

  __syncthreads();                                     // the output tile reuses the stages
  store_tile<BM, BN, WTM, WTN, TM, TN, RAGGED_M, T, 2 * STAGE_BYTES, OUT, FMT != kNvfp4>(
      acc, smem, factors, nv_mul, W.bias != nullptr, M, N, m0, n0, wave_m, wave_n, tm_cnt, tid, 1.0f,
      tile_m * tiles_n + tile_n, out);
}

// ------------------------------------------------------------------------ INT scale prepass
// One wave per row of scales (see int_row_scale).  blockIdx.y: the operand (a launch for each took 2.5 us more than one for
// both).
struct ScalePrep {
  const float* s;
  uint16_t* h;
  float* mul;
  int rows;
  const uint8_t* codes;      // MARK only
};
// MARK: rows with codes outside -4 .. 3 are marked (see wide_codes_tile)
template <bool MARK>
__global__ __launch_bounds__(256) void int_scale_prep_kernel(ScalePrep a, ScalePrep w, int groups, float Q, int K) {
  const ScalePrep& o = blockIdx.y ? w : a;
  const float* __restrict__ s = o.s;
  uint16_t* __restrict__ h_out = o.h;
  float* __restrict__ mul_out = o.mul;
  const int rows = o.rows;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= rows) return;
  const float* sr = s + (int64_t)row * groups;
  // 16-byte pieces of the row's codes; the first on its way with the scales
  const uint4* cr = MARK ? reinterpret_cast<const uint4*>(o.codes + (int64_t)row * (K / 2)) : nullptr;
  uint4 first = make_uint4(0u, 0u, 0u, 0u);
  if (MARK && lane < K / 32) first = cr[lane];
  float mx = 0.0f;
  for (int g = lane; g < groups; g += 64) mx = fmaxf(mx, int_group_max(sr[g], Q));
  const RowScale scale = int_row_scale(wave_max(mx));
  for (int g = lane; g < groups; g += 64) h_out[(int64_t)row * groups + g] = int_scale_unit(sr[g], Q, scale.down);
  bool marked = false;
  if constexpr (MARK) {
    uint32_t wide = wide_codes(first.x) | wide_codes(first.y) | wide_codes(first.z) | wide_codes(first.w);
#pragma unroll 4
    for (int c = lane + 64; c < K / 32; c += 64) {
      const uint4 v = cr[c];
      wide |= wide_codes(v.x) | wide_codes(v.y) | wide_codes(v.z) | wide_codes(v.w);
    }
    marked = __any((wide & kWideBits) != 0);
  }
  if (lane == 0) mul_out[row] = marked ? -(scale.up / Q) : scale.up / Q;
}

// ------------------------------------------------------------------------ INT scale form check
// The product folds the group maximum h = bf16_rne(s * Q) into its fp16 operands instead of the stored
// scale s, which is the same number only if s = fl32(h / Q) -- true for what the quantizers of this
// library write from bf16 inputs, not for arbitrary fp32 scales.  This kernel counts the scales that
// are not of that form (and the negative or non-finite ones).
__global__ __launch_bounds__(256) void check_int_scales_kernel(const float* __restrict__ s, int64_t n, float Q,
                                                               unsigned long long* __restrict__ bad) {
  unsigned int mine = 0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const float v = s[i];
    const float h = as_f32(f32_to_bf16_rne(v * Q) << 16);
    const bool ok = v >= 0.0f && v <= 3.0e38f && div_const(h, Q, 1.0f / Q) == v;
    mine += ok ? 0u : 1u;
  }
  // wave total, one atomic per wave
  for (int off = 32; off >= 1; off >>= 1) mine += (unsigned int)__shfl_xor((int)mine, off, kWave);
  if ((threadIdx.x & 63) == 0 && mine) atomicAdd(bad, (unsigned long long)mine);
}

__global__ void zero_u64_kernel(unsigned long long* p) { *p = 0ull; }

int run_check_int_scales(pq_format fmt, int group, const void* scales, int64_t rows, int64_t K, int64_t* bad_count,
                         void* ws, hipStream_t st) {
  const int64_t n = rows * (K / group);
  unsigned long long* bad = (unsigned long long*)ws;
  hipLaunchKernelGGL(zero_u64_kernel, dim3(1), dim3(1), 0, st, bad);
  int64_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(check_int_scales_kernel, dim3((unsigned)blocks), dim3(256), 0, st, (const float*)scales, n,
                     qmax_of((int)fmt), bad);
  int rc = check_hip(hipGetLastError(), "check_int_scales_kernel");
  if (rc) return rc;
  double* h = pinned_doubles(1);
  if (!h) return fail(PQ_ERR_HIP, "pq_qgemm_check_int_scales: no pinned host memory");
  if ((rc = check_hip(hipMemcpyAsync(h, bad, 8, hipMemcpyDeviceToHost, st), "copy count"))) return rc;
  if ((rc = check_hip(hipStreamSynchronize(st), "hipStreamSynchronize"))) return rc;
  unsigned long long c;
  memcpy(&c, h, 8);
  *bad_count = (int64_t)c;
  return PQ_OK;
}

// ------------------------------------------------------------------------ host side
struct GemmWs {
  uint16_t* a_h;
  uint16_t* w_h;
  float* a_mul;
  float* w_mul;
};

static size_t carve_gemm(void* base, pq_format fmt, int group, int64_t M, int64_t N, int64_t K,
                         GemmWs* w) {
  if (fmt == PQ_FMT_NVFP4) return 0;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off = align_up(off + bytes, 256);
    return o;
  };
  size_t o_ah = take((size_t)M * (K / group) * 2);
  size_t o_wh = take((size_t)N * (K / group) * 2);
  size_t o_am = take((size_t)M * 4);
  size_t o_wm = take((size_t)N * 4);
  if (w) {
    char* b = (char*)base;
    w->a_h = (uint16_t*)(b + o_ah);
    w->w_h = (uint16_t*)(b + o_wh);
    w->a_mul = (float*)(b + o_am);
    w->w_mul = (float*)(b + o_wm);
  }
  return off;
}

size_t qgemm_workspace_bytes(pq_format fmt, int group, int64_t M, int64_t N, int64_t K) {
  return carve_gemm(nullptr, fmt, group, M, N, K, nullptr);
}

template <int FMT, int G, int BM, int BN, int WGM, int WGN, int OUT>
static int launch_gemm(const OperandView& A, const OperandView& W, int M, int N, int K, const Outputs& out,
                       hipStream_t st) {
  constexpr int T = WGM * WGN * 64;
  constexpr size_t shmem = 2 * (size_t)((BM * 2 + T - 1) / T * (T / 2) + BN) * kRowBytes + kFactorBytes<BM, BN>;
  auto kern = qgemm_kernel<FMT, G, BM, BN, WGM, WGN, OUT>;
  static std::atomic<uint64_t> raised{0};
  if (int rc = allow_lds(reinterpret_cast<const void*>(kern), shmem, raised, "hipFuncSetAttribute(qgemm_kernel)")) return rc;
  int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  int64_t n_tiles = (int64_t)tiles_m * tiles_n;
  if (n_tiles > 0x7FFFFFFF) return fail(PQ_ERR_SHAPE, "too many output tiles");
  hipLaunchKernelGGL(kern, dim3((unsigned)n_tiles, out.problems), dim3(T), shmem, st, A, W, M, N, K, out, tiles_m, tiles_n);
  return check_hip(hipGetLastError(), "qgemm_kernel");
}

template <int FMT, int G, int OUT>
static int pick_tile(const OperandView& A, const OperandView& W, int M, int N, int K, const Outputs& out,
                     int choice, hipStream_t st) {
  if constexpr (G <= 32) {                             // larger groups: pq_qgemm_group.hip
    if (choice == kTile256) return launch_gemm<FMT, G, 256, 256, 2, 4, OUT>(A, W, M, N, K, out, st);
    if (choice == kTile224) return launch_gemm<FMT, G, 224, 256, 2, 4, OUT>(A, W, M, N, K, out, st);
  }
  return launch_gemm<FMT, G, 128, 128, 2, 2, OUT>(A, W, M, N, K, out, st);
}

template <int FMT, int G>
static int launch_views_fg(const OperandView& A, const OperandView& W, int M, int N, int K, const Outputs& out, int tile,
                           hipStream_t st) {
  if (out.kind == kOutF32) return pick_tile<FMT, G, kOutF32>(A, W, M, N, K, out, tile, st);
  if (out.kind == kOutDiff) return pick_tile<FMT, G, kOutDiff>(A, W, M, N, K, out, tile, st);
  return pick_tile<FMT, G, kOutBf16>(A, W, M, N, K, out, tile, st);
}

// the product kernel on two operand views (any mix of layouts)
int launch_qgemm_views(pq_format fmt, int group, const OperandView& A, const OperandView& W, int64_t M,
                       int64_t N, int64_t K, const Outputs& out, int tile, hipStream_t st) {
  if (tile >= kTileSplit32)
    return launch_qgemm_split(fmt, group, A, W, (int)M, (int)N, (int)K, out, tile, st);
  // groups of 64 and more in large tiles: the codes go to the matrix unit as they are
  if (fmt != PQ_FMT_NVFP4 && group != 32 && tile != kTile128)
    return launch_qgemm_group(fmt, group, A, W, (int)M, (int)N, (int)K, out, tile, st);
#define PQ_ARGS A, W, (int)M, (int)N, (int)K, out, tile, st
  if (fmt == PQ_FMT_NVFP4) return launch_views_fg<kNvfp4, 16>(PQ_ARGS);
  if (fmt == PQ_FMT_INT4 || fmt == PQ_FMT_INT3) {      // the nibbles of both unpack alike
    switch (group) {
      case 32: return launch_views_fg<kInt4, 32>(PQ_ARGS);
      case 64: return launch_views_fg<kInt4, 64>(PQ_ARGS);
      case 128: return launch_views_fg<kInt4, 128>(PQ_ARGS);
      case 256: return launch_views_fg<kInt4, 256>(PQ_ARGS);
    }
  }
#undef PQ_ARGS
  return fail(PQ_ERR_FORMAT, "unsupported (format, group) = (%d, %d)", (int)fmt, group);
}

// Operands in the row-major layout of the quantizers.  NVFP4 scales are read in place; INT
// scales go through the per-row normalisation pass into `ws` first (phases & 1), the product
// (phases & 2) then reads that working copy.
int run_qgemm(pq_format fmt, int group, const uint8_t* a_codes, const void* a_scales,
              const float* a_ts, const uint8_t* w_codes, const void* w_scales, const float* w_ts,
              int64_t M, int64_t N, int64_t K, void* y, int64_t ldy, bool out_f32, int phases,
              void* ws, hipStream_t st) {
  OperandView A{a_codes, K / 2, 32, nullptr, 0, 2, nullptr, 0};
  OperandView W{w_codes, K / 2, 32, nullptr, 0, 2, nullptr, 0};
  if (fmt == PQ_FMT_NVFP4) {
    A.scales = (const uint8_t*)a_scales;
    W.scales = (const uint8_t*)w_scales;
    A.sc_row = W.sc_row = K / 16;
    A.mul = a_ts;
    W.mul = w_ts;
  } else {
    if (fmt != PQ_FMT_INT4 && fmt != PQ_FMT_INT3)
      return fail(PQ_ERR_FORMAT, "unsupported (format, group) = (%d, %d)", (int)fmt, group);
    GemmWs G;
    carve_gemm(ws, fmt, group, M, N, K, &G);
    const float Q = qmax_of((int)fmt);
    const int tile = choose_tile(fmt, group, M, N, K);
    if (phases == 3 && split_takes_raw_scales(fmt, group, tile, M, N, K)) {
      A.scales = (const uint8_t*)a_scales;
      W.scales = (const uint8_t*)w_scales;
      A.sc_row = W.sc_row = (K / group) * 4;
      A.sc_step = W.sc_step = 4;
      const Output out{out_f32 ? kOutF32 : kOutBf16, y, ldy, nullptr, false};
      return launch_qgemm_split_raw(fmt, group, A, W, (int)M, (int)N, (int)K,
                                    RawOutput{out, {Q, G.a_h, G.w_h, G.a_mul, G.w_mul}}, tile, st);
    }
    const bool mark = phases == 3 && fmt == PQ_FMT_INT3 && group != 32;
    if (phases & 1) {
      const int64_t most = M > N ? M : N;
      hipLaunchKernelGGL(mark ? int_scale_prep_kernel<true> : int_scale_prep_kernel<false>,
                         dim3((unsigned)((most + 3) / 4), 2), dim3(256), 0, st,
                         ScalePrep{(const float*)a_scales, G.a_h, G.a_mul, (int)M, a_codes},
                         ScalePrep{(const float*)w_scales, G.w_h, G.w_mul, (int)N, w_codes},
                         (int)(K / group), Q, (int)K);
      int rc = check_hip(hipGetLastError(), "int_scale_prep_kernel");
      if (rc) return rc;
    }
    A.scales = (const uint8_t*)G.a_h;
    W.scales = (const uint8_t*)G.w_h;
    A.sc_row = W.sc_row = (K / group) * 2;
    A.mul = G.a_mul;
    W.mul = G.w_mul;
    A.mul_stride = W.mul_stride = 1;
    A.marked = W.marked = mark;
  }
  if (!(phases & 2)) return PQ_OK;
  return launch_qgemm_views(fmt, group, A, W, M, N, K, Outputs{{out_f32 ? kOutF32 : kOutBf16, y, ldy, nullptr, false}},
                            choose_tile(fmt, group, M, N, K), st);
}

}  // namespace pq
