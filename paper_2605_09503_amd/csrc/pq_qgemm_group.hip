// Low-bit GEMM for the integer formats on the 8- and 4-bit matrix instructions (paper Eq. 8):
//     Y[m, n] = sum_g (sa[m, g] sw[n, g]) I_g[m, n],   I_g[m, n] = sum_{k in g} a[m, k] w[n, k]
//
// The codes go to the matrix unit as they are and the scales stay outside:
//   P = v_mfma_f32_32x32x64_f8f6f4 of 64 codes of k (no accumulator input): the exact integer I_g in fp32,
//       |I_g| <= 64 * 49, times a power of two;
//   S = v_mfma_f32_32x32x8_f16 with a single non-zero k: the outer product of the two scale columns, 8-bit
//       times 8-bit significands (the fp16 scale units of the operand layout), exact in fp32;
//   acc += P * S, one fused multiply-add per output and group on the vector unit.
// The only roundings are those fused multiply-adds, one per 64 k (a product of fp16 operands that carry
// their scale accumulates with a rounding per matrix instruction, four per 64 k), and the epilogue's.
//
// Code formats.  INT4: E4M3, whose subnormals and first binade are the integers 0..15 times 2^-9, so a byte
// sign << 7 | |z| is z 2^-9 exactly (all sixteen nibbles, -8 included).  INT3: E2M1, where 0, .5, 1, 1.5, 2
// are the codes 0..4, so a nibble sign << 3 | |z| is z / 2 exactly for |z| <= 4.
//
// What bounds it.  Beside matrix instructions a vector instruction takes an issue slot of 4.2 cycles and the matrix
// instruction one more; what does not fit into the matrix cycles is added to them (measured with two waves a SIMD: 6
// beside a 32-cycle one 34 to 39 cycles, 8 44, 16 69 to 80).  A 32 x 32 x 64 block takes:
//   fp16 operands that carry their scale (pq_qgemm.hip)   128 matrix cycles + 16 vector instructions (the unpack)
//   8-bit codes (here, INT4)                          64 + 32 matrix cycles + 31 (16 multiply-adds, 11 of unpack)
//   4-bit codes (here, INT3)                          32 + 32 matrix cycles + 23 (16 multiply-adds, 4 of unpack)
// and the 8- and 4-bit instructions draw less power: the chip holds 2.3 GHz here and 1.9 GHz there.  Forming S
// on the vector unit instead would be 16 more instructions a block.  Measured, us and TFLOP/s (before: fp16):
//   INT3 g64   4608 x 3072 x 3072     76 -> 49  (1.77 PFLOP/s)    8192 x 12288 x 3072   490 -> 307 (2.01)
//   INT4 g64   4608 x 3072 x 3072     80 -> 66  (1.31)            8192 x 12288 x 3072   515 -> 411 (1.50)
//   INT4 g64   4608 x 3072 x 12288   295 -> 234 (1.49)
// Groups of 32 would need two half-empty matrix products and two scale products a block, 128 matrix cycles again,
// and 32 multiply-adds: 510 us against 477 on INT3 8192 x 12288 x 3072, so they stay on the fp16 kernel, as do NVFP4's
// groups of 16.  Issuing the next block's matrix instructions before this block's multiply-adds needs 16 to 32
// more registers than a wave has: spilled, and slower (INT4 75 -> 95 us).
//
// Structure as in pq_qgemm.hip: one workgroup per output tile, every thread unpacks one 32-code slice of
// each operand per 64-wide step, global loads run ahead in registers.  LDS holds four steps, so that the one
// barrier of a step can sit in its middle: the first fragments of the next step are fetched before the current
// one ends, and no wave starts a step waiting for LDS (with three stages and the barrier at the end of the step
// 89 us instead of 78 on INT4 4608 x 3072 x 3072).
#include "pq_qgemm_common.h"

namespace pq {

// FP4: E2M1 codes (INT3), else E4M3 (INT4).  Groups are a multiple of 64 (2^g_shift).  WIDE: how codes that E2M1 does
// not hold are found.
template <bool FP4, int BM, int BN, int WGM, int WGN, int OUT, int WIDE>
__global__ __launch_bounds__(WGM* WGN * 64) void qgemm_group_kernel(OperandView A, OperandView W, int M, int N,
                                                                    int K, int g_shift, KernelOutput<OUT> out, int tiles_m,
                                                                    int tiles_n) {
  if constexpr (OUT == kOutDiff) enter_problem(A, W, out);
  constexpr int T = WGM * WGN * 64;
  constexpr int WTM = (BM + WGM * 32 - 1) / (WGM * 32) * 32, WTN = BN / WGN;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  constexpr int TM_LAST = (BM - (WGM - 1) * WTM) / 32;
  constexpr bool RAGGED_M = TM_LAST != TM;
  constexpr int SL = BN * 2 / T;
  static_assert(BN * 2 % T == 0 && (BM * 2 + T - 1) / T == SL, "whole slices per thread, as many for A as for W");
  static_assert(BM % 32 == 0 && WTN % 32 == 0 && TM_LAST >= 1 && TM_LAST <= TM, "wave tile");
  static_assert(!RAGGED_M || (WGM == 2 && WGN == 4), "the uneven split is laid out for 2 x 4 waves");
  constexpr int A_ROWS = SL * (T / 2);
  constexpr int RB = FP4 ? 32 : 64;                    // LDS bytes of a row: 64 codes
  constexpr int NP = RB / 32;                          // 16-byte pieces of a 32-code slice
  constexpr int A_CODES = 0, W_CODES = A_ROWS * RB, A_SC = W_CODES + BN * RB, W_SC = A_SC + A_ROWS * 4;
  constexpr int STAGE_BYTES = W_SC + BN * 4, STAGES = 4;
  constexpr int OUT_BYTES = OUT != kOutBf16 ? 0 : BM * (BN * 2 + 16);
  constexpr int SMEM_BYTES = STAGES * STAGE_BYTES > OUT_BYTES ? STAGES * STAGE_BYTES : OUT_BYTES;
  constexpr int FMT_SEL = FP4 ? 4 : 0;                 // operand format field of the matrix instruction

  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

  int tile_m, tile_n;
  assign_tile(tiles_m, tiles_n, tile_m, tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * BN;

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wave_m = RAGGED_M ? ((wave >> 2) ^ wave) & 1 : wave % WGM;
  const int wave_n = RAGGED_M ? wave >> 1 : wave / WGM;
  const int tm_cnt = RAGGED_M ? __builtin_amdgcn_readfirstlane(wave_m == WGM - 1 ? TM_LAST : TM) : TM;

  // loader: this thread owns tile row tid / 2, k offset 32 * (tid & 1), of both operands
  const int ld_row = tid >> 1, ld_half = tid & 1;
  static_assert(SL == 1, "a thread's two slices are of one row of either tile");
  // addresses: a uniform part (the tile, the step) and a 32-bit offset inside the tile.  Rows past the last re-read it: what
  // they give is not stored.
  const int a_row = min(ld_row, M - 1 - m0), w_row = min(ld_row, N - 1 - n0);
  const uint32_t a_coff = (uint32_t)a_row * (uint32_t)A.code_row + ld_half * 16u;
  const uint32_t w_coff = (uint32_t)w_row * (uint32_t)W.code_row + ld_half * 16u;
  const uint8_t* a_codes = A.codes + (int64_t)m0 * A.code_row;
  const uint8_t* w_codes = W.codes + (int64_t)n0 * W.code_row;
  // of the two threads of a row the lower half's loads and stores the scale of A's, the other that of W's
  const uint8_t* sc_row = ld_half ? W.scales + (int64_t)(n0 + w_row) * W.sc_row : A.scales + (int64_t)(m0 + a_row) * A.sc_row;
  const int sc_step = ld_half ? W.sc_step : A.sc_step;
  // Loads never leave the operand and never branch (a branch in the loop would split its schedule): a step past the last
  // re-reads the last.  What it holds does not matter: its scales are stored as zero.  (K is a multiple of 64 here.)
  const int ksteps = K / kBK;
  auto load_codes = [&](const uint8_t* codes, uint32_t coff, int code_step, int step) {
    const int st = min(step, ksteps - 1);                             // uniform
    return *reinterpret_cast<const uint4*>(codes + (int64_t)st * code_step + coff);
  };
  auto load_a = [&](int step, uint4& r) { r = load_codes(a_codes, a_coff, A.code_step, step); };
  auto load_w = [&](int step, uint4& r, uint32_t& sc) {
    r = load_codes(w_codes, w_coff, W.code_step, step);
    const int unit = (min(step, ksteps - 1) * kBK) >> g_shift;        // uniform
    sc = *reinterpret_cast<const uint16_t*>(sc_row + (int64_t)unit * sc_step);
  };

  // Placement of a row's 16-byte pieces: rotated by the row so that the 16 rows that share a 256-byte line
  // of banks in a fragment read use different banks.
  auto piece_at = [&](int row, int piece) {
    const int f = FP4 ? (row >> 3) & 1 : (row >> 2) & 3;
    return row * RB + ((piece ^ f) << 4);
  };
  // piece 0 of this thread's slice; piece 1 is 16 bytes beside it, on the side the rotation says (stages and
  // tiles start at multiples of 32 bytes: an exclusive or)
  const int st_off = piece_at(ld_row, ld_half * NP);
  // A row's scale has a word of its own in LDS and one thread that loads and stores it, after the step's codes: a load, a store and
  // their offsets less in every step than with both scales in both threads of a row, as halves of words.  us, so -> now: INT4 g64
  // 8192 x 12288 x 3072 423 -> 411, INT3 320 -> 307, 4608 x 3072 x 3072 (224 rows) 66.0 -> 66.3 and 49.9 -> 49.1; stored ahead of the
  // codes INT4's 224-row tile 67.1.  (Bank conflicts, 0.8 of the active LDS cycles, are as many as before.)
  const int sc_at = (ld_half ? W_SC : A_SC) + ld_row * 4;
  auto put_scale = [&](int st, uint32_t sc, bool ok) {
    *reinterpret_cast<uint32_t*>(smem + st + sc_at) = sc & (ok ? ~0u : 0u);
  };
  uint32_t wide = 0;
  // 16-byte piece c of a slice: unpacked and stored
  auto put_piece = [&](const uint4& s, int codes, int c) {
    const uint32_t d[4] = {s.x, s.y, s.z, s.w};
    if constexpr (FP4) {
      if constexpr (WIDE == kWideCodes) wide |= wide_codes(d[0]) | wide_codes(d[1]) | wide_codes(d[2]) | wide_codes(d[3]);
      *reinterpret_cast<uint4*>(smem + (codes + st_off)) =
          make_uint4(e2m1_nibbles(d[0]), e2m1_nibbles(d[1]), e2m1_nibbles(d[2]), e2m1_nibbles(d[3]));
    } else {
      uint32_t o[4];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const uint32_t v = c == 0 ? d[e] : d[2 + e];
        o[2 * e] = e4m3_bytes(v & 0x0F0F0F0Fu, (v >> 3) & 0x01010101u);
        o[2 * e + 1] = e4m3_bytes((v >> 4) & 0x0F0F0F0Fu, (v >> 7) & 0x01010101u);
      }
      *reinterpret_cast<uint4*>(smem + ((codes + st_off) ^ (c << 4))) = make_uint4(o[0], o[1], o[2], o[3]);
    }
  };

  // fragment addresses inside a stage: the row of a tile is lane % 32, its half of the 64 k lane / 32; tiles
  // lie 32 rows apart, which leaves the placement of the pieces unchanged
  const int frag_row = lane & 31, frag_half = lane >> 5;
  const int x_base = A_CODES + piece_at(wave_m * WTM + frag_row, frag_half * NP);
  const int w_base = W_CODES + piece_at(wave_n * WTN + frag_row, frag_half * NP);
  const int xs_base = A_SC + (wave_m * WTM + frag_row) * 4;
  const int ws_base = W_SC + (wave_n * WTN + frag_row) * 4;

  struct Frag {
    int4v v[NP];
  };
  auto read_frag = [&](int base, int stage, int tile) {
    Frag f;
#pragma unroll
    for (int c = 0; c < NP; ++c)
      f.v[c] = *reinterpret_cast<const int4v*>(smem + ((stage + base) ^ (c << 4)) + tile * 32 * RB);
    return f;
  };
  auto read_scale = [&](int base, int stage, int tile) {
    return *reinterpret_cast<const uint32_t*>(smem + stage + base + tile * 128);
  };
  auto operand = [&](const Frag& f) {
    if constexpr (FP4) return (int8v){f.v[0].x, f.v[0].y, f.v[0].z, f.v[0].w, 0, 0, 0, 0};
    else return (int8v){f.v[0].x, f.v[0].y, f.v[0].z, f.v[0].w, f.v[NP - 1].x, f.v[NP - 1].y, f.v[NP - 1].z, f.v[NP - 1].w};
  };
  float16_t acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  // Slices on their way from memory: two steps' worth with 4-bit codes; with 8-bit codes, whose fragments take
  // twice the registers, one step's, reloaded as soon as it is unpacked.
  constexpr int RS = FP4 ? 2 : 1;
  uint4 raw_a[2], raw_w[2];                            // [1] is dead after the prologue for RS = 1
  uint32_t raw_sc[2];

  // ---- prologue: stages 0 and 1 <- steps 0 and 1, raw[0] <- step 2 (raw[1] <- step 3)
  load_a(0, raw_a[0]);
  load_w(0, raw_w[0], raw_sc[0]);
  load_a(1, raw_a[1]);
  load_w(1, raw_w[1], raw_sc[1]);
  float* const factors = reinterpret_cast<float*>(smem + SMEM_BYTES + (WIDE == kWideCodes ? T / 16 : 0));
  {
    Factors<BM, BN, T, true> f;
    f.load(A, W, M, N, m0, n0);
    f.put(factors);
  }
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int st = p * STAGE_BYTES;
    const bool k_ok = p * kBK < K;
#pragma unroll
    for (int c = 0; c < NP; ++c) {
      put_piece(raw_a[p], st + A_CODES, c);
      put_piece(raw_w[p], st + W_CODES, c);
    }
    put_scale(st, raw_sc[p], k_ok);
    if (p < RS) {
      load_a(p + 2, raw_a[p]);
      load_w(p + 2, raw_w[p], raw_sc[p]);
    }
  }
  __syncthreads();

  const float16_t zero = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f,
                          0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
  Frag wf[TN], xf[2];
  uint32_t sw[TN], sx[2];
#pragma unroll
  for (int i = 0; i < TN; ++i) {
    wf[i] = read_frag(w_base, 0, i);
    sw[i] = read_scale(ws_base, 0, i);
  }
  xf[0] = read_frag(x_base, 0, 0);
  sx[0] = read_scale(xs_base, 0, 0);
  int st_cur = 0;                                      // byte offset of the stage being multiplied
  auto stage_after = [&](int st, int n) {
    const int v = st + n * STAGE_BYTES;
    return v >= STAGES * STAGE_BYTES ? v - STAGES * STAGE_BYTES : v;
  };

  // X0: which of the two activation fragments tile row 0 of this step sits in
  auto body = [&](auto Pc, auto TMc, auto X0c, int s) {
    constexpr int P = decltype(Pc)::value;
    constexpr int TMW = decltype(TMc)::value;
    constexpr int X0 = decltype(X0c)::value;
    constexpr int NT = TMW * TN;                       // tiles of this wave
    constexpr int NW = 2 * NP;                         // pieces to unpack, all in the first half of the tiles
    uint4 &ra = raw_a[P % RS], &rw = raw_w[P % RS];
    uint32_t& rsc = raw_sc[P % RS];
    const int st_next = stage_after(st_cur, 1), st_put = stage_after(st_cur, 2);
    const bool k_ok = (s + 2) * kBK < K;

    half4v swz[TN];
#pragma unroll
    for (int i = 0; i < TN; ++i) swz[i] = scale_operand(frag_half == 0 ? sw[i] : 0u);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int j = t / TN, i = t % TN;
      const int8v xo = operand(xf[(X0 + j) & 1]);
      const float16_t sc = __builtin_amdgcn_mfma_f32_32x32x8f16(swz[i], scale_operand(sx[(X0 + j) & 1]), zero, 0, 0, 0);
      const float16_t p = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(operand(wf[i]), xo, zero, FMT_SEL, FMT_SEL, 0, 0, 0, 0);
      // while the matrix unit works: fragments to come, and this thread's share of step s + 2
      if (i == 0) {
        const int nx = (X0 + j + 1) & 1;
        if (j + 1 < TMW) {
          xf[nx] = read_frag(x_base, st_cur, j + 1);
          sx[nx] = read_scale(xs_base, st_cur, j + 1);
        } else {
          xf[nx] = read_frag(x_base, st_next, 0);
          sx[nx] = read_scale(xs_base, st_next, 0);
        }
      }
      if (j == TMW - 1) {                              // the last use of weight fragment i in this step
        wf[i] = read_frag(w_base, st_next, i);
        sw[i] = read_scale(ws_base, st_next, i);
      }
#pragma unroll
      for (int u = 0; u < NW; ++u) {
        if (u * (NT / 2) / NW != t) continue;
        const int c = u % NP;
        if (u < NP) {
          put_piece(ra, st_put + A_CODES, c);
        } else {
          put_piece(rw, st_put + W_CODES, c);
        }
        if (u == NW - 1) put_scale(st_put, rsc, k_ok);
        if (u == NP - 1) load_a(s + 2 + RS, ra);
        if (u == NW - 1) load_w(s + 2 + RS, rw, rsc);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = __builtin_fmaf(p[r], sc[r], acc[i][j][r]);
      __builtin_amdgcn_sched_barrier(0);
      // One barrier a step, in its middle.  It publishes the stage written above, whose first fragments are
      // read at the end of the next step; and the stage written in the next step was last read in the step
      // before this one.
      if (t == NT / 2) {
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    st_cur = st_next;
  };

  // two steps per trip (the register sets are compile-time constants); an odd step count runs one extra step
  // on zero scales
  if (!RAGGED_M || tm_cnt == TM) {
    for (int s = 0; s < ksteps; s += 2) {
      body(IntC<0>{}, IntC<TM>{}, IntC<0>{}, s);
      body(IntC<1>{}, IntC<TM>{}, IntC<TM & 1>{}, s + 1);
    }
  } else {
    for (int s = 0; s < ksteps; s += 2) {
      body(IntC<0>{}, IntC<TM_LAST>{}, IntC<0>{}, s);
      body(IntC<1>{}, IntC<TM_LAST>{}, IntC<TM_LAST & 1>{}, s + 1);
    }
  }

  __syncthreads();                                     // the output tile reuses the stages
  uint32_t marks = 0;
  if constexpr (WIDE == kWideMarks) marks = tile_marks<BM, BN>(factors);
  store_tile<BM, BN, WTM, WTN, TM, TN, RAGGED_M, T, SMEM_BYTES, OUT, true>(
      acc, smem, factors, 0.0f, W.bias != nullptr, M, N, m0, n0, wave_m, wave_n, tm_cnt, tid,
      FP4 ? 4.0f : 262144.0f, tile_m * tiles_n + tile_n, out);
  if constexpr (WIDE != kWideNone) {                   // here, where the accumulators are dead
    const bool any = WIDE == kWideMarks ? __any((int)marks < 0) != 0
                                        : any_wide<T / 64>(wide, reinterpret_cast<int*>(smem + SMEM_BYTES));
    if (any) {
      __threadfence();                                 // what the waves stored has arrived
      __syncthreads();
      wide_codes_tile<BM, BN, T / 64, 1, OUT>(A, W, M, N, K, g_shift, m0, n0, out);
    }
  }
}

template <bool FP4, int BM, int BN, int WGM, int WGN, int OUT, int WIDE>
static int launch_group(const OperandView& A, const OperandView& W, int M, int N, int K, int g_shift, const Outputs& out,
                        hipStream_t st) {
  constexpr int T = WGM * WGN * 64;
  constexpr int A_ROWS = (BM * 2 + T - 1) / T * (T / 2);
  constexpr size_t stages = 4 * (size_t)(A_ROWS + BN) * ((FP4 ? 32 : 64) + 4);
  constexpr size_t tile_bytes = OUT != kOutBf16 ? 0 : (size_t)BM * (BN * 2 + 16);
  constexpr size_t shmem = (stages > tile_bytes ? stages : tile_bytes) + (WIDE == kWideCodes ? WGM * WGN * 4 : 0) + kFactorBytes<BM, BN>;
  auto kern = qgemm_group_kernel<FP4, BM, BN, WGM, WGN, OUT, WIDE>;
  static std::atomic<uint64_t> raised{0};
  if (int rc = allow_lds(reinterpret_cast<const void*>(kern), shmem, raised, "hipFuncSetAttribute(qgemm_group_kernel)")) return rc;
  const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  const int64_t n_tiles = (int64_t)tiles_m * tiles_n;
  if (n_tiles > 0x7FFFFFFF) return fail(PQ_ERR_SHAPE, "too many output tiles");
  hipLaunchKernelGGL(kern, dim3((unsigned)n_tiles, out.problems), dim3(T), shmem, st, A, W, M, N, K, g_shift, out, tiles_m,
                     tiles_n);
  return check_hip(hipGetLastError(), "qgemm_group_kernel");
}

template <bool FP4, int OUT, int WIDE>
static int group_tile(const OperandView& A, const OperandView& W, int M, int N, int K, int g_shift, const Outputs& out,
                      int choice, hipStream_t st) {
  if (choice == kTile256) return launch_group<FP4, 256, 256, 2, 4, OUT, WIDE>(A, W, M, N, K, g_shift, out, st);
  return launch_group<FP4, 224, 256, 2, 4, OUT, WIDE>(A, W, M, N, K, g_shift, out, st);
}

// INT4 and INT3 with groups of 64, 128 or 256, large tiles
int launch_qgemm_group(pq_format fmt, int group, const OperandView& A, const OperandView& W, int M, int N, int K,
                       const Outputs& out, int choice, hipStream_t st) {
  const int g_shift = group == 64 ? 6 : group == 128 ? 7 : 8;
#define PQ_ARGS (A, W, M, N, K, g_shift, out, choice, st)
  if (fmt == PQ_FMT_INT4) {
    if (out.kind == kOutF32) return group_tile<false, kOutF32, kWideNone> PQ_ARGS;
    if (out.kind == kOutDiff) return group_tile<false, kOutDiff, kWideNone> PQ_ARGS;
    return group_tile<false, kOutBf16, kWideNone> PQ_ARGS;
  }
  // the selection (kOutDiff) multiplies what it quantized itself
  if (out.kind == kOutDiff) return group_tile<true, kOutDiff, kWideNone> PQ_ARGS;
  if (A.marked && W.marked) {
    if (out.kind == kOutF32) return group_tile<true, kOutF32, kWideMarks> PQ_ARGS;
    return group_tile<true, kOutBf16, kWideMarks> PQ_ARGS;
  }
  if (out.kind == kOutF32) return group_tile<true, kOutF32, kWideCodes> PQ_ARGS;
  return group_tile<true, kOutBf16, kWideCodes> PQ_ARGS;
#undef PQ_ARGS
}

}  // namespace pq
