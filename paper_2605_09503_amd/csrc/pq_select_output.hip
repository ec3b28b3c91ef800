// Permutation selection with the layer-output error as the calibration metric -- the other reading
// of "the candidate with the smallest quantization error on the calibration data" (paper Sec. 3.3):
//     E_out(pi) = sum_b ||X_b W^T - Q(X_b P) Q(P^T W)^T||^2 / sum_b ||X_b W^T||^2        (Eq. 8)
// The candidate orders are those of pq_select_perm (joint score, Eq. 9, alpha grid).  The quantized
// product runs through the forward path (gathering quantizer straight into the operand layout, product kernel whose
// epilogue keeps the squared difference to the unquantized product instead of a result); the unquantized product
// comes from a plain bf16 MFMA kernel below, which also sums its squares.  Every sum has a fixed order.
//
// The batches of a call stand one below the other as the rows of one product, and several candidate orders share a
// launch (see plan_of): one quantizer launch for all their operands, one product launch whose grid holds all their
// tiles.  With a product launch for each order and batch, 1024 x 3072 x 3072 with two batches of INT4 took 14
// products of 30 us, none of which filled the chip with large tiles, and 21 quantizer launches: 715 us, now 381
// (NVFP4 659 -> 379, INT3 g64 3 x 700 x 1000 x 1152 354 -> 128, INT4 g64 4 x 4608 x 3072 x 3072 3.73 -> 2.98 ms).
#include <string.h>

#include <algorithm>

#include "pq_qgemm_common.h"

namespace pq {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

constexpr int kRefRows = 128;                 // rows of an output tile
constexpr int kRefStep = 64;                  // K elements per step
constexpr int kRefRowBytes = kRefStep * 2;

// Columns of the tile and stages of LDS: 128 with two, two workgroups a unit, or 192 with three and one.
template <int TN>
struct RefTile {
  static constexpr int cols = TN * 64, stages = TN == 2 ? 2 : 3;
  static constexpr int stage_bytes = (kRefRows + cols) * kRefRowBytes, lds_bytes = stages * stage_bytes;
  static constexpr int loads = (kRefRows + cols) / 32;      // 16-byte pieces of a step, per thread
};

// 16 bytes a lane from memory into LDS, 1 KB a wave from byte `to` on, without a register in between: by a 64-bit address, or
// by a uniform base and an offset.  m0, an operand, holds `to`.  The wait for them is ref_wait's.
__device__ __forceinline__ void load_to_lds(uint32_t to, const uint8_t* from) {
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"{m0}"(to), "v"(from) : "memory");
}
__device__ __forceinline__ void load_to_lds(uint32_t to, const uint8_t* base, uint32_t offset) {
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"{m0}"(to), "v"(offset), "s"(base) : "memory");
}
// all but the last N loads of this wave have arrived and its LDS reads are done; then the workgroup meets
template <int N>
__device__ __forceinline__ void ref_wait() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// Y[m, n] = sum_k X[m, k] W[n, k], bf16 inputs, fp32 accumulation (v_mfma_f32_32x32x16_bf16), fp32 output, and the
// tile's sum of squares (+)= to sq.  X: the rows of all batches.  Four waves of 64 x 32 TN; K % 32 == 0.  The pieces of a step go
// from memory straight into LDS, one or two steps ahead: through registers their stores took more of the LDS pipe than the
// reads did.  Rows of 128 bytes lie unpadded, a row's 16-byte pieces permuted by (row / 2) % 8, so that the 16 rows of
// a read have a piece of every bank.  One barrier a step: behind it the step has arrived, and the stage of the step before is
// free.  us, 128 x 128 tiles through registers -> now: 2048 x 3072 x 3072 69 -> 49
// (128 x 192, one a unit), 3072 x 3072 x 1024 44 -> 41; 0.77 us a step of 64 and 12 to 16 that do not depend on K (a store of rows through LDS
// and a start at another k for every tile: the same).
template <int TN>
__global__ __launch_bounds__(256) void ref_gemm_kernel(RowBatches xs, const uint16_t* __restrict__ w,
                                                       int M, int N, int K, float* __restrict__ y, int64_t ldy,
                                                       double* __restrict__ sq, int add, int tiles_m, int tiles_n) {
  using R = RefTile<TN>;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave_m = wave & 1, wave_n = wave >> 1;
  int tile_m, tile_n;
  assign_tile(tiles_m, tiles_n, tile_m, tile_n);
  const int m0 = tile_m * kRefRows, n0 = tile_n * R::cols;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds;

  // loader: the wave's load i takes rows 8 (4 i + wave) .. + 7 of an operand, lane l the piece that belongs at place l % 8 of
  // row l / 8
  constexpr int XL = kRefRows / 32, WL = R::cols / 32;
  const uint8_t* x_at[XL];
  uint32_t w_at[WL];
  const int ld_row = lane >> 3;
  auto piece_of = [&](int row) { return (lane & 7) ^ ((row >> 1) & 7); };
#pragma unroll
  for (int i = 0; i < XL; ++i) {
    const int row = 8 * (4 * i + wave) + ld_row, m = min(m0 + row, M - 1), batch = m / (int)xs.rows;
    const uint16_t* x = xs.p[0];
#pragma unroll
    for (int b = 1; b < kMaxMomentBatches; ++b) x = batch == b ? xs.p[b] : x;      // an index by lane would go through scratch
    x_at[i] = reinterpret_cast<const uint8_t*>(x + (int64_t)(m - batch * (int)xs.rows) * K) + piece_of(row) * 16;
  }
#pragma unroll
  for (int i = 0; i < WL; ++i) {
    const int row = 8 * (4 * i + wave) + ld_row;
    w_at[i] = (uint32_t)min(row, N - 1 - n0) * ((uint32_t)K * 2u) + piece_of(row) * 16;
  }
  const uint8_t* w_tile = reinterpret_cast<const uint8_t*>(w + (int64_t)n0 * K);
  const int steps = (K + kRefStep - 1) / kRefStep;
  const bool half_last = K % kRefStep != 0;
  // a step past the last re-reads the last and is not multiplied; the missing upper half of a last step of 32 re-reads the lower
  auto load = [&](int step, int stage) {
    const int st = min(step, steps - 1);               // uniform
    const uint32_t to = lds0 + stage * R::stage_bytes;
    const bool half = half_last && st == steps - 1;    // uniform
    const int64_t at = (int64_t)st * kRefRowBytes;
#pragma unroll
    for (int i = 0; i < XL; ++i) {
      const int row = 8 * (4 * i + wave) + ld_row;
      load_to_lds(to + (4 * i + wave) * 1024, x_at[i] + (at - (half && piece_of(row) >= 4 ? 64 : 0)));
    }
#pragma unroll
    for (int i = 0; i < WL; ++i) {
      const int row = 8 * (4 * i + wave) + ld_row;
      load_to_lds(to + kRefRows * kRefRowBytes + (4 * i + wave) * 1024, w_tile + at, w_at[i] - (half && piece_of(row) >= 4 ? 64u : 0u));
    }
  };

  const int frag_row = lane & 31, frag_half = lane >> 5;
  int piece[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) piece[kk] = ((kk * 2 + frag_half) ^ ((frag_row >> 1) & 7)) * 16;
  const int x_row = (wave_m * 64 + frag_row) * kRefRowBytes;
  const int w_row = (kRefRows + wave_n * (R::cols / 2) + frag_row) * kRefRowBytes;

  float16_t acc[TN][2];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  // The fragments of 16 k are read while those before them are multiplied, the first of a step behind the barrier that stands
  // before the last 16 k of the step before: there that step's stage is read and free for the step R::stages on.
  bf16x8_t xf[2][2], wf[2][TN];
  auto read = [&](int set, int stage, int kk) {
    const unsigned char* at = lds + stage * R::stage_bytes + piece[kk];
#pragma unroll
    for (int j = 0; j < 2; ++j) xf[set][j] = *reinterpret_cast<const bf16x8_t*>(at + x_row + j * 32 * kRefRowBytes);
#pragma unroll
    for (int i = 0; i < TN; ++i) wf[set][i] = *reinterpret_cast<const bf16x8_t*>(at + w_row + i * 32 * kRefRowBytes);
  };
  auto multiply = [&](int set) {
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[set][i], xf[set][j], acc[i][j], 0, 0, 0);
  };
#pragma unroll
  for (int p = 0; p < R::stages; ++p) load(p, p);
  ref_wait<(R::stages - 1) * R::loads>();
  read(0, 0, 0);
  int stage = 0;
  for (int s = 0; s < K / kRefStep; ++s) {
#pragma unroll
    for (int kk = 0; kk < 3; ++kk) {
      read((kk + 1) & 1, stage, kk + 1);
      multiply(kk & 1);
    }
    ref_wait<(R::stages - 2) * R::loads>();
    load(s + R::stages, stage);
    stage = stage + 1 == R::stages ? 0 : stage + 1;
    read(0, stage, 0);
    multiply(1);
  }
  if (half_last) {                                     // uniform
    read(1, stage, 1);
    multiply(0);
    multiply(1);
  }
  ref_wait<0>();                                       // the sums below take the stages
  // lane holds, per 32 x 32 block, column m = lane % 32 and rows n = 8 (r / 4) + 4 (lane / 32) + r % 4
  double s2 = 0.0;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int m = m0 + wave_m * 64 + j * 32 + frag_row;
    if (m >= M) continue;
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int n = n0 + wave_n * (R::cols / 2) + i * 32 + q * 8 + frag_half * 4;
        float* yo = y + (int64_t)m * ldy + n;
        const float v[4] = {acc[i][j][q * 4], acc[i][j][q * 4 + 1], acc[i][j][q * 4 + 2], acc[i][j][q * 4 + 3]};
        if (n + 3 < N) *reinterpret_cast<float4*>(yo) = make_float4(v[0], v[1], v[2], v[3]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (n + e < N) {
            if (n + 3 >= N) yo[e] = v[e];
            s2 = fma((double)v[e], (double)v[e], s2);
          }
        }
      }
  }
  store_diff(s2, reinterpret_cast<double*>(lds), 256, tile_m * tiles_n + tile_n, Output{kOutDiff, sq, 0, nullptr, add != 0});
}

int64_t ref_tiles(int64_t M, int64_t N, int cols) { return ((M + kRefRows - 1) / kRefRows) * ((N + cols - 1) / cols); }

// Columns of the reference product's tile: the ones whose fullest unit has the fewer outputs; the smaller where it is the same,
// and where K is short: two workgroups run beside each other, and one's stores, which do not get shorter with K, hide behind
// the other's loads (4592 x 6500 x 96 32.5 us, with 192 columns 40.2; 6208 x 4909 x 64 31.5, 38.9).  Over 1056 random shapes (64 to
// 12288 rows and columns, K 64 to 12288) the better tile's time is missed by 0.2 % in the mean, by more than 5 % for 18 of them, at most
// 11 % (873 x 9820 x 9312: three rounds of the small tile 259 us, two of the large one 233); without the line in K 0.4 %, 39, 24 %.
int ref_cols(int64_t M, int64_t N, int64_t K) {
  const auto fullest = [&](int cols) { return (ref_tiles(M, N, cols) + 255) / 256 * cols; };
  return K >= 8 * kRefStep && fullest(192) < fullest(128) ? 192 : 128;
}

template <int TN>
int launch_ref(const RowBatches& x, const void* w, int64_t M, int64_t N, int64_t K, float* y, int64_t ldy, double* sq, bool add,
               hipStream_t st) {
  using R = RefTile<TN>;
  static std::atomic<uint64_t> raised{0};
  auto kern = ref_gemm_kernel<TN>;
  if (int rc = allow_lds(reinterpret_cast<const void*>(kern), R::lds_bytes, raised, "hipFuncSetAttribute(ref_gemm_kernel)")) return rc;
  const int64_t tiles_m = (M + kRefRows - 1) / kRefRows, tiles_n = (N + R::cols - 1) / R::cols;
  if (tiles_m * tiles_n > UINT32_MAX / 256) return fail(PQ_ERR_SHAPE, "too many output tiles");     // more threads than a grid holds
  hipLaunchKernelGGL(kern, dim3((unsigned)(tiles_m * tiles_n)), dim3(256), R::lds_bytes, st, x, (const uint16_t*)w, (int)M, (int)N,
                     (int)K, y, ldy, sq, add, (int)tiles_m, (int)tiles_n);
  return check_hip(hipGetLastError(), "ref_gemm_kernel");
}

// sums[c] = sum of the tiles of candidate c (c < n_cand), sums[den_at] = sum of the reference's tiles; fixed order
__global__ __launch_bounds__(256) void tile_sums_kernel(const double* __restrict__ num, int64_t num_stride, int64_t tiles,
                                                        const double* __restrict__ den, int64_t den_tiles, int n_cand,
                                                        int den_at, double* __restrict__ sums) {
  __shared__ double red[4];
  const bool is_den = (int)blockIdx.x == n_cand;
  const double* p = is_den ? den : num + (int64_t)blockIdx.x * num_stride;
  const int64_t n = is_den ? den_tiles : tiles;
  double s = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += 256) s += p[i];
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) sums[is_den ? den_at : (int)blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// moved[j] = number of positions where candidate j differs from the identity; ts: the two tensor scales
__global__ __launch_bounds__(1024) void moved_kernel(const int32_t* __restrict__ cands, int K, double* __restrict__ moved,
                                                     float* __restrict__ ts, float act_ts, float w_ts) {
  const int j = blockIdx.x;
  if (j == 0 && threadIdx.x == 0) {
    ts[0] = act_ts;
    ts[1] = w_ts;
  }
  __shared__ int red[16];
  int c = 0;
  for (int i = threadIdx.x; i < K; i += 1024) c += __popcll(__ballot(cands[(int64_t)j * K + i] != i));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    int all = 0;
    for (int w = 0; w < 16; ++w) all += red[w];
    moved[j] = (double)all;
  }
}

constexpr int kMaxCandOut = PQ_MAX_ALPHAS + 1;
constexpr int kNumSums = kMaxCandOut + 1 + PQ_MAX_ALPHAS;

// How a call is cut into launches: `stack` batches stand one below the other, `orders` orders are quantized and multiplied
// together.  As many as give the product three rounds of its largest tile over the 256 units: from there on a launch
// more costs less than the operands' memory (an order's operands take 4.25 bits an element).
struct Plan {
  int stack, orders;
};
Plan plan_of(int64_t M, int64_t N, int n_batches) {
  constexpr int64_t kTiles = 3 * 256;
  auto tiles = [&](int64_t rows) { return ((rows + 255) / 256) * ((N + 255) / 256); };
  const int64_t most = n_batches < kMaxMomentBatches ? n_batches : kMaxMomentBatches;
  const int64_t stack = std::min(most, (kTiles + tiles(M) - 1) / tiles(M));
  const int64_t all = tiles(stack * M);
  return Plan{(int)stack, (int)std::min<int64_t>(kMaxCandOut, (kTiles + all - 1) / all)};
}
constexpr Plan kOneByOne{1, 1};

struct OutWs {
  double* keys;
  int32_t* cands;
  int32_t* rank;
  float* y_ref;        // [n_batches][M][ldn]
  uint8_t* x_op;       // [orders] operands of stack * M rows
  uint8_t* w_op;       // [orders]
  float* ts;           // [2] activation and weight tensor scale
  double* num;         // [kMaxCandOut][tiles of the product, at most out_tiles(stack * M, N)]
  double* den;         // [tiles of the reference product]
  double* sums;        // [kMaxCandOut] numerators, [1] denominator, [PQ_MAX_ALPHAS] moved counts
};

// tiles of the smallest size any product kernel takes
size_t out_tiles(int64_t M, int64_t N) { return (size_t)((M + 31) / 32) * ((N + 31) / 32); }
size_t carve_out(void* base, const Plan& p, pq_format fmt, int group, int64_t M, int64_t N, int64_t K, int n_batches,
                 OutWs* w) {
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off = align_up(off + bytes, 256);
    return o;
  };
  const int64_t ldn = (N + 7) / 8 * 8, rows = p.stack * M;
  const size_t o_keys = take((size_t)PQ_MAX_ALPHAS * K * 8);
  const size_t o_cands = take((size_t)PQ_MAX_ALPHAS * K * 4);
  const size_t o_rank = take((size_t)PQ_MAX_ALPHAS * K * 4);
  const size_t o_ref = take((size_t)n_batches * M * ldn * 4);
  const size_t o_xop = take(p.orders * operand_bytes(fmt, group, rows, K));
  const size_t o_wop = take(p.orders * operand_bytes(fmt, group, N, K));
  const size_t o_ts = take(2 * sizeof(float));
  const size_t o_num = take(kMaxCandOut * out_tiles(rows, N) * 8);
  const size_t o_den = take((size_t)ref_tiles(rows, N, 128) * 8);         // the smaller tile
  const size_t o_sums = take((size_t)kNumSums * 8);
  if (w) {
    char* b = (char*)base;
    w->keys = (double*)(b + o_keys);
    w->cands = (int32_t*)(b + o_cands);
    w->rank = (int32_t*)(b + o_rank);
    w->y_ref = (float*)(b + o_ref);
    w->x_op = (uint8_t*)(b + o_xop);
    w->w_op = (uint8_t*)(b + o_wop);
    w->ts = (float*)(b + o_ts);
    w->num = (double*)(b + o_num);
    w->den = (double*)(b + o_den);
    w->sums = (double*)(b + o_sums);
  }
  return off;
}

}  // namespace

size_t select_output_workspace_bytes(pq_format fmt, int group, int64_t M, int64_t N, int64_t K, int n_batches) {
  return carve_out(nullptr, plan_of(M, N, n_batches), fmt, group, M, N, K, n_batches, nullptr);
}
size_t select_output_least_workspace_bytes(pq_format fmt, int group, int64_t M, int64_t N, int64_t K, int n_batches) {
  return carve_out(nullptr, kOneByOne, fmt, group, M, N, K, n_batches, nullptr);
}

// The plan of a call with such a workspace: where it does not hold the operands of plan_of, as many orders as fit, dealt
// evenly over the launches, then (an order at a time) as many batches.  INT4 g64, 8 x 64 rows, 12288 x 12288 weights, seven
// orders in one launch take 614 MB, four 363, one 113 (a batch at a time 109).
static Plan plan_within(pq_format fmt, int group, int64_t M, int64_t N, int64_t K, int n_batches, int n_cand, size_t ws_bytes) {
  Plan p = plan_of(M, N, n_batches);
  p.orders = std::min(p.orders, n_cand);
  const auto fits = [&] { return carve_out(nullptr, p, fmt, group, M, N, K, n_batches, nullptr) <= ws_bytes; };
  if (fits()) return p;
  while (p.orders > 1 && !fits()) --p.orders;
  while (p.stack > 1 && !fits()) --p.stack;
  const int launches = (n_cand + p.orders - 1) / p.orders;
  p.orders = (n_cand + launches - 1) / launches;
  return p;
}
// One tile and number of waves for the whole call, those of a full launch: a last launch of fewer batches adds its sums
// to the first slots of the same ones, and equal orders have equal sums whichever launch takes them.
static int tile_of_call(pq_format fmt, int group, int64_t M, int64_t N, int64_t K, const Plan& plan) {
  return choose_tile(fmt, group, plan.stack * M, N, K, plan.orders);
}

void select_output_plan(pq_format fmt, int group, int64_t M, int64_t N, int64_t K, int n_batches, int n_alpha, size_t ws_bytes,
                        pq_output_plan* out) {
  const Plan plan = plan_within(fmt, group, M, N, K, n_batches, n_alpha + 1, ws_bytes);
  const int tile = tile_of_call(fmt, group, M, N, K, plan);
  out->batches = plan.stack;
  out->orders = plan.orders;
  tile_size(tile, &out->tile_m, &out->tile_n);
  out->tile_waves = tile_waves(tile);
}

int run_select_output(pq_format fmt, int group, const double* act_sumsq, const double* w_sumsq, int64_t K,
                      const void* const* x_calib, int n_batches, int64_t M, const void* w, int64_t N,
                      float act_ts, float w_ts, const double* alphas, int n_alpha, double tau,
                      int32_t* perm_out, pq_select_report* report, void* ws, size_t ws_bytes, hipStream_t st) {
  const int n_cand = n_alpha + 1;              // candidate 0 is the original order
  const Plan plan = plan_within(fmt, group, M, N, K, n_batches, n_cand, ws_bytes);
  OutWs W;
  carve_out(ws, plan, fmt, group, M, N, K, n_batches, &W);
  const int64_t ldn = (N + 7) / 8 * 8;
  const int stack = plan.stack, orders = plan.orders;
  if (stack * M * 32 > 0x7FFFFFFF || N * 32 > 0x7FFFFFFF) return fail(PQ_ERR_SHAPE, "too many rows for the panel layout");
  int rc;
  if ((rc = launch_candidate_orders(act_sumsq, w_sumsq, K, alphas, n_alpha, W.keys, W.rank, W.cands, st))) return rc;
  hipLaunchKernelGGL(moved_kernel, dim3(n_alpha), dim3(1024), 0, st, W.cands, (int)K, W.sums + kMaxCandOut + 1, W.ts, act_ts,
                     w_ts);
  if ((rc = check_hip(hipGetLastError(), "moved_kernel"))) return rc;

  // batches b0 .. b0 + stack - 1 as rows
  auto rows_from = [&](int b0, int64_t* rows) {
    const int nb = std::min(stack, n_batches - b0);
    RowBatches x;
    for (int b = 0; b < kMaxMomentBatches; ++b) x.p[b] = (const uint16_t*)x_calib[b0 + (b < nb ? b : 0)];
    x.rows = M;
    *rows = nb * M;
    return x;
  };
  // the unquantized products, once
  const int cols = ref_cols(stack * M, N, K);
  for (int b0 = 0; b0 < n_batches; b0 += stack) {
    int64_t rows;
    const RowBatches x = rows_from(b0, &rows);
    float* y = W.y_ref + (size_t)b0 * M * ldn;
    rc = cols == 192 ? launch_ref<3>(x, w, rows, N, K, y, ldn, W.den, b0 > 0, st) : launch_ref<2>(x, w, rows, N, K, y, ldn, W.den, b0 > 0, st);
    if (rc) return rc;
  }

  const int64_t most_rows = stack * M;
  const int tile = tile_of_call(fmt, group, M, N, K, plan);
  const size_t num_stride = out_tiles(stack * M, N);
  const size_t w_next = operand_bytes(fmt, group, N, K);
  const RowBatches w_rows = {{(const uint16_t*)w}, N};
  for (int c0 = 0; c0 < n_cand; c0 += orders) {
    const int n = std::min(orders, n_cand - c0);
    for (int b0 = 0; b0 < n_batches; b0 += stack) {
      int64_t rows;
      const RowBatches x = rows_from(b0, &rows);
      const size_t x_next = operand_bytes(fmt, group, rows, K);
      // the tensor scale of the weights does not depend on the order: the caller's value is used
      const PanelJob xj{x, rows, W.x_op, x_next, W.ts}, wj{w_rows, b0 ? 0 : N, W.w_op, w_next, W.ts + 1};
      if ((rc = launch_quantize_rows_panel(fmt, group, xj, wj, K, W.cands, c0, n, st))) return rc;
      Outputs out{{kOutDiff, W.num + (size_t)c0 * num_stride, ldn, W.y_ref + (size_t)b0 * M * ldn, b0 > 0}};
      out.a_next = x_next;
      out.w_next = w_next;
      out.y_next = (int64_t)num_stride;
      out.problems = (unsigned)n;
      const OperandView A = panel_view(fmt, group, W.x_op, rows, K, W.ts), B = panel_view(fmt, group, W.w_op, N, K, W.ts + 1);
      if ((rc = launch_qgemm_views(fmt, group, A, B, rows, N, K, out, tile, st))) return rc;
    }
  }
  hipLaunchKernelGGL(tile_sums_kernel, dim3((unsigned)(n_cand + 1)), dim3(256), 0, st, W.num, (int64_t)num_stride,
                     qgemm_tiles(tile, most_rows, N), W.den, ref_tiles(most_rows, N, cols), n_cand, kMaxCandOut, W.sums);
  if ((rc = check_hip(hipGetLastError(), "tile_sums_kernel"))) return rc;

  double* h = pinned_doubles(kNumSums);
  if (!h) return fail(PQ_ERR_HIP, "pq_select_perm_output_error: no pinned host memory for the sums");
  if ((rc = check_hip(hipMemcpyAsync(h, W.sums, (size_t)kNumSums * 8, hipMemcpyDeviceToHost, st), "copy sums")))
    return rc;
  if ((rc = check_hip(hipStreamSynchronize(st), "hipStreamSynchronize"))) return rc;

  const double den = h[kMaxCandOut];
  double E[kMaxCandOut];
  for (int c = 0; c < n_cand; ++c) E[c] = h[c] / den;
  int best = 0;
  for (int j = 1; j < n_alpha; ++j)
    if (E[1 + j] < E[1 + best]) best = j;         // first minimum: smallest alpha on ties
  const double e_orig = E[0], e_best = E[1 + best];
  const bool accepted = h[kMaxCandOut + 1 + best] != 0.0 && e_orig > 0.0 && ((e_orig - e_best) / e_orig > tau);
  memset(report, 0, sizeof(*report));
  report->accepted = accepted ? 1 : 0;
  report->alpha_index = best;
  report->e_orig = e_orig;
  report->e_best = e_best;
  for (int j = 0; j < n_alpha; ++j) report->e_cand[j] = E[1 + j];
  report->sum_x2 = den;            // here: ||X W^T||^2 over the calibration batches
  report->sum_w2 = 0.0;
  return launch_emit_order(accepted ? W.cands + (int64_t)best * K : nullptr, perm_out, K, st);
}

}  // namespace pq
