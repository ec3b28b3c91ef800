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
// products of 30 us, none of which filled the chip with large tiles, and 21 quantizer launches: 715 us, now 406
// (NVFP4 659 -> 423, INT3 g64 3 x 700 x 1000 x 1152 354 -> 131, INT4 g64 4 x 4608 x 3072 x 3072 3.73 -> 3.14 ms).
#include <string.h>

#include <algorithm>

#include "pq_qgemm_common.h"

namespace pq {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

constexpr int kRefTile = 128;                 // output tile edge
constexpr int kRefStep = 64;                  // K elements per step
constexpr int kRefRowBytes = kRefStep * 2 + 16;   // padded LDS row, as in pq_qgemm.hip
constexpr int kRefStage = 2 * kRefTile * kRefRowBytes;

// Y[m, n] = sum_k X[m, k] W[n, k], bf16 inputs, fp32 accumulation (v_mfma_f32_32x32x16_bf16), fp32 output, and the
// tile's sum of squares (+)= to sq.  X: the rows of all batches.  128 x 128 tile, four waves of 64 x 64; K % 32 == 0.  A
// step's pieces are loaded two steps before they are multiplied and stored, a step before, into the other of two stages: one
// barrier a step.  Bound by the stores and reads of the stages, which a tile of this size has two of for each product: 70 us
// for 2048 x 3072 x 3072 (a launch for each half, loaded one step ahead: 48 us each).
__global__ __launch_bounds__(256) void ref_gemm_kernel(RowBatches xs, const uint16_t* __restrict__ w,
                                                       int M, int N, int K, float* __restrict__ y, int64_t ldy,
                                                       double* __restrict__ sq, int add) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wave_m = wave & 1, wave_n = wave >> 1;
  const int m0 = blockIdx.x * kRefTile, n0 = blockIdx.y * kRefTile;
  // loader: 128 rows x 128 bytes per operand; thread t takes piece t % 8 of rows t / 8 + 32 i
  const int ld_row = tid >> 3, ld_piece = tid & 7;
  const uint16_t *xr[4], *wr[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = min(m0 + ld_row + 32 * i, M - 1), batch = m / (int)xs.rows;
    const uint16_t* x = xs.p[0];
#pragma unroll
    for (int b = 1; b < kMaxMomentBatches; ++b) x = batch == b ? xs.p[b] : x;      // an index by lane would go through scratch
    xr[i] = x + (int64_t)(m - batch * (int)xs.rows) * K + ld_piece * 8;
    wr[i] = w + (int64_t)min(n0 + ld_row + 32 * i, N - 1) * K + ld_piece * 8;
  }
  const int st = ld_row * kRefRowBytes + ld_piece * 16;
  const int frag_row = lane & 31, frag_half = lane >> 5;
  struct Pieces {
    int4v a[4], w[4];
  };
  // a step past the last re-reads the start of the rows and is not multiplied; the upper half of a last step of 32 is zero
  auto load = [&](int k0, Pieces& p) {
    const int k = k0 + ld_piece * 8 < K ? k0 : -ld_piece * 8;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      p.a[i] = *reinterpret_cast<const int4v*>(xr[i] + k);
      p.w[i] = *reinterpret_cast<const int4v*>(wr[i] + k);
    }
  };
  auto put = [&](unsigned char* stage, int k0, const Pieces& p) {
    const bool ok = k0 + ld_piece * 8 < K;
    const int4v zero = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      *reinterpret_cast<int4v*>(stage + st + 32 * i * kRefRowBytes) = ok ? p.a[i] : zero;
      *reinterpret_cast<int4v*>(stage + kRefTile * kRefRowBytes + st + 32 * i * kRefRowBytes) = ok ? p.w[i] : zero;
    }
  };

  float16_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  Pieces pieces[2];
  load(0, pieces[0]);
  load(kRefStep, pieces[1]);
  put(lds, 0, pieces[0]);
  __syncthreads();
  // step k0, in stage P; pieces[P ^ 1] holds the next one, if there is one, pieces[P] is free
  auto turn = [&](auto Pc, int k0, auto last) {
    constexpr int P = decltype(Pc)::value;
    constexpr bool kMore = !decltype(last)::value;
    if constexpr (kMore) load(k0 + 2 * kRefStep, pieces[P]);
    const unsigned char* a_t = lds + P * kRefStage;
    const unsigned char* w_t = a_t + kRefTile * kRefRowBytes;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      bf16x8_t xf[2], wf[2];
#pragma unroll
      for (int j = 0; j < 2; ++j)
        xf[j] = *reinterpret_cast<const bf16x8_t*>(a_t + (wave_m * 64 + j * 32 + frag_row) * kRefRowBytes +
                                                   (kk * 2 + frag_half) * 16);
#pragma unroll
      for (int i = 0; i < 2; ++i)
        wf[i] = *reinterpret_cast<const bf16x8_t*>(w_t + (wave_n * 64 + i * 32 + frag_row) * kRefRowBytes +
                                                   (kk * 2 + frag_half) * 16);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[i], xf[j], acc[i][j], 0, 0, 0);
    }
    if constexpr (kMore) {
      put(lds + (P ^ 1) * kRefStage, k0 + kRefStep, pieces[P ^ 1]);
      __syncthreads();
    }
  };
  // two steps a trip, then an odd last one (a step of zeros in its place: 2048 x 3072 x 64 19.6 us, so 16.9; x 320 20.6, 18.8)
  int k0 = 0;
  for (; k0 + kRefStep < K; k0 += 2 * kRefStep) {
    turn(IntC<0>{}, k0, IntC<0>{});
    turn(IntC<1>{}, k0 + kRefStep, IntC<0>{});
  }
  if (k0 < K) turn(IntC<0>{}, k0, IntC<1>{});
  // lane holds, per 32 x 32 block, column m = lane % 32 and rows n = 8 (r / 4) + 4 (lane / 32) + r % 4
  double s2 = 0.0;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int m = m0 + wave_m * 64 + j * 32 + frag_row;
    if (m >= M) continue;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int n = n0 + wave_n * 64 + i * 32 + q * 8 + frag_half * 4;
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
  store_diff(s2, reinterpret_cast<double*>(lds), 256, blockIdx.y * gridDim.x + blockIdx.x,
             Output{kOutDiff, sq, 0, nullptr, add != 0});
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
size_t ref_tiles(int64_t M, int64_t N) {
  return (size_t)((M + kRefTile - 1) / kRefTile) * ((N + kRefTile - 1) / kRefTile);
}

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
  const size_t o_den = take(ref_tiles(rows, N) * 8);
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
  static std::atomic<uint64_t> raised{0};
  if ((rc = allow_lds(reinterpret_cast<const void*>(ref_gemm_kernel), 2 * kRefStage, raised,
                      "hipFuncSetAttribute(ref_gemm_kernel)")))
    return rc;
  for (int b0 = 0; b0 < n_batches; b0 += stack) {
    int64_t rows;
    const RowBatches x = rows_from(b0, &rows);
    const dim3 grid((unsigned)((rows + kRefTile - 1) / kRefTile), (unsigned)((N + kRefTile - 1) / kRefTile));
    hipLaunchKernelGGL(ref_gemm_kernel, grid, dim3(256), 2 * kRefStage, st, x, (const uint16_t*)w, (int)rows, (int)N, (int)K,
                       W.y_ref + (size_t)b0 * M * ldn, ldn, W.den, b0 > 0);
  }
  if ((rc = check_hip(hipGetLastError(), "ref_gemm_kernel"))) return rc;

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
                     qgemm_tiles(tile, most_rows, N), W.den, (int64_t)ref_tiles(most_rows, N), n_cand, kMaxCandOut, W.sums);
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
