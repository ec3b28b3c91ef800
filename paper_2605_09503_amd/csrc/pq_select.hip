// Permutation selection (paper Sec. 3.3): joint second-moment score (Eq. 9), descending sort
// (Prop. 1), calibration error of every candidate order, alpha search and acceptance rule.
//
// Kernels
//   block_order_kernel  key[j][i] = alpha_j ln Sa[i] + (1 - alpha_j) ln Sw[i], fp64, all j in one
//                     launch (a term whose weight is zero is skipped), in order inside every block of 256 channels.
//   rank_merge_kernel / rank_scatter_kernel
//                     stable descending sort: rank(i) = #{j : key_j > key_i or (key_j == key_i and
//                     j < i)}, from the sorted blocks by bisection, integer counts added atomically
//                     (deterministic); perm[rank(i)] = i, and which orders repeat an earlier one (or the
//                     original order): those are evaluated once.  K <= 65536.
//   quant_error_kernel a workgroup stages a few rows in LDS at a time; for every candidate order
//                     their channels are gathered from LDS (one read serves all resident rows),
//                     quantized with the same lane-cooperative quantizer as the runtime kernels,
//                     and the squared error of the dequantized values accumulated in fp64 (NVFP4:
//                     from exact fp32 group sums).  HBM traffic is one read of the tensor for all
//                     candidates.
//   select_tail_kernel fixed-order sums of the per-wave partial errors, of the moments and of the
//                     moved-channel counts (deterministic), one launch.
// The final argmin / acceptance decision is a handful of scalar operations and runs on the host.
#include <string.h>

#include <atomic>
#include <type_traits>

#include "pq_device.h"
#include "pq_host.h"

namespace pq {

constexpr int kMaxCand = PQ_MAX_ALPHAS + 1;   // identity + candidates

struct AlphaList {
  double a[PQ_MAX_ALPHAS];
};

// The stable descending sort, in blocks of 256 channels: block_order_kernel puts every block in order, and the rank
// of a channel is its place there plus, for every other block, the number of keys that sort before its own, found by
// bisection.  Both passes, six orders: 24 us at K = 12288 and 10.8 at K = 3072, where a pass for the keys and one that
// counts against all K of them took 63 and 12.
constexpr int kSortBlock = 256;
constexpr int kMergeBlocks = 4;    // blocks a workgroup of the merging pass bisects in
constexpr int kSortShares = 4;     // threads that share a channel's comparisons inside its block

// Workgroup (x, y): the keys of channel block x for alpha_y,
//     key[i] = alpha ln Sa[i] + (1 - alpha) ln Sw[i],
// in descending order, equal keys in ascending channel order: keys into key[y], channels into order[y].  With
// sa == nullptr the keys are in key[] already.  Also clears what the passes after it add to.
__global__ __launch_bounds__(kSortBlock * kSortShares) void block_order_kernel(const double* __restrict__ sa,
                                                                 const double* __restrict__ sw, int64_t K,
                                                                 AlphaList alphas, double* __restrict__ keys,
                                                                 int32_t* __restrict__ order, int32_t* __restrict__ rank,
                                                                 uint32_t* __restrict__ differs) {
  __shared__ double tile[kSortBlock];
  __shared__ int before_of[kSortShares][kSortBlock];
  const int t = threadIdx.x % kSortBlock, share = threadIdx.x / kSortBlock;      // share: uniform over a wave
  const int64_t i0 = (int64_t)blockIdx.x * kSortBlock, i = i0 + t;
  double* key = keys + (int64_t)blockIdx.y * K;
  double k = -__builtin_inf();
  if (share == 0) {
    if (differs && i == 0) differs[blockIdx.y] = 0u;  // rank_scatter_kernel ORs into it
    if (i < K) {
      if (sa) {
        const double alpha = alphas.a[blockIdx.y];
        k = 0.0;
        if (alpha != 0.0) k += alpha * log(sa[i]);
        if (alpha != 1.0) k += (1.0 - alpha) * log(sw[i]);
      } else {
        k = key[i];
      }
      if (!(k == k)) k = -__builtin_inf();            // no number (a negative statistic): last, and still an order
      rank[(int64_t)blockIdx.y * K + i] = 0;          // the merging pass adds to it
    }
    tile[t] = k;                                      // past K: after every channel, and after its equals
  }
  __syncthreads();
  k = tile[t];
  int before = 0;
  constexpr int kShare = kSortBlock / kSortShares;
#pragma unroll 16
  for (int j = share * kShare; j < (share + 1) * kShare; ++j) {
    // without short-circuit evaluation: no branches
    const double kj = tile[j];
    const int gt = kj > k ? 1 : 0, eq = kj == k ? 1 : 0, earlier = j < t ? 1 : 0;
    before += gt | (eq & earlier);
  }
  before_of[share][t] = before;
  __syncthreads();
  if (share == 0 && i < K) {
    int at = 0;
#pragma unroll
    for (int q = 0; q < kSortShares; ++q) at += before_of[q][t];
    key[i0 + at] = k;
    order[(int64_t)blockIdx.y * K + i0 + at] = (int32_t)i;
  }
}

// Workgroup (x, y, z): for the channels of block x of order z, how many keys of blocks y * kMergeBlocks ... sort before
// theirs, added to rank[z] (integer atomics: the sum does not depend on order).  A key of an earlier block sorts
// before an equal one, of a later block after it.  The channel's place in its own block is added along with it.
__global__ __launch_bounds__(kSortBlock) void rank_merge_kernel(const double* __restrict__ keys,
                                                                const int32_t* __restrict__ order, int K, int n_blocks,
                                                                int32_t* __restrict__ rank) {
  __shared__ double tile[kMergeBlocks][kSortBlock];
  const double* key = keys + (int64_t)blockIdx.z * K;
  const int b0 = blockIdx.y * kMergeBlocks;
  // a missing key is the smallest there is: never greater than another, and only the last block, which no channel
  // comes after, is short
#pragma unroll
  for (int b = 0; b < kMergeBlocks; ++b) {
    const int j = (b0 + b) * kSortBlock + threadIdx.x;
    tile[b][threadIdx.x] = j < K ? key[j] : -__builtin_inf();
  }
  __syncthreads();
  const int i = blockIdx.x * kSortBlock + threadIdx.x;
  if (i >= K) return;
  const double ki = key[i];
  int before[kMergeBlocks];
#pragma unroll
  for (int b = 0; b < kMergeBlocks; ++b) before[b] = 0;
  // in step with each other, so that the chains of reads overlap
#pragma unroll
  for (int half = kSortBlock / 2; half >= 1; half >>= 1) {
#pragma unroll
    for (int b = 0; b < kMergeBlocks; ++b) {
      const double kj = tile[b][before[b] + half - 1];
      const bool ahead = b0 + b < (int)blockIdx.x ? kj >= ki : kj > ki;
      before[b] += ahead ? half : 0;
    }
  }
  int sum = 0;
#pragma unroll
  for (int b = 0; b < kMergeBlocks; ++b) {
    // the bisection stops short of the block's last key
    const double kj = tile[b][kSortBlock - 1];
    const bool all = before[b] == kSortBlock - 1 && (b0 + b < (int)blockIdx.x ? kj >= ki : kj > ki);
    const int n = before[b] + (all ? 1 : 0);
    sum += b0 + b >= n_blocks ? 0 : b0 + b == (int)blockIdx.x ? (int)threadIdx.x : n;
  }
  atomicAdd(&rank[(int64_t)blockIdx.z * K + order[(int64_t)blockIdx.z * K + i]], sum);
}

// perm[z][rank(i)] = i; with offs, also the LDS byte offset of channel i's slot in the error evaluation
// (slot i + i / 8, slot_bytes each) at the same position.  With differs: which candidate orders repeat an earlier one.
// Candidate 0 is the original order, candidate 1 + j the order of alpha_j.  differs[j] collects a bit per earlier candidate
// c <= j that differs from order j somewhere (integer OR: no order dependence).  Two orders are the same when every
// channel has the same rank in both, so the ranks tell, and no pass over the finished orders is needed: six orders, K =
// 3072 3.5 us, with that pass 2.5 + 4.9; K = 12288 6.7, 5.1 + 6.2.  differs[] is zeroed by block_order_kernel, which runs
// before on the same stream.
__global__ __launch_bounds__(256) void rank_scatter_kernel(const int32_t* __restrict__ rank, int K,
                                                           int32_t* __restrict__ perms,
                                                           int32_t* __restrict__ offs, int slot_bytes,
                                                           uint32_t* __restrict__ differs) {
  const int i = blockIdx.x * 256 + threadIdx.x, j = blockIdx.y;
  const bool ok = i < K;
  const int at = ok ? rank[(int64_t)j * K + i] : i;
  if (ok) {
    perms[(int64_t)j * K + at] = i;
    if (offs) offs[(int64_t)j * K + at] = (i + (i >> 3)) * slot_bytes;
  }
  if (differs) {
    // all loads, then a bit of the wave at a time, then one atomic a workgroup: they are served one after the other
    __shared__ uint32_t wave_bits[4];
    uint32_t d = at != i ? 1u : 0u;                          // bit 0: the original order
    if (ok) {
#pragma unroll 4
      for (int e = 0; e < j; ++e) d |= (rank[(int64_t)e * K + i] != at ? 1u : 0u) << (1 + e);
    }
    uint32_t bits = 0u;
    for (int b = 0; b <= j; ++b) bits |= (__any((d >> b) & 1u) ? 1u : 0u) << b;
    if ((threadIdx.x & 63) == 0) wave_bits[threadIdx.x >> 6] = bits;
    __syncthreads();
    if (threadIdx.x == 0) {
      bits = wave_bits[0] | wave_bits[1] | wave_bits[2] | wave_bits[3];
      if (bits) atomicOr(&differs[j], bits);
    }
  }
}
// the first candidate with the same order as candidate c (c itself if none before it)
__device__ __forceinline__ int first_same_order(const uint32_t* __restrict__ differs, int c) {
  if (c == 0) return 0;
  const uint32_t bits = differs[c - 1];
  int first = c;
  for (int e = c - 1; e >= 0; --e)
    if (!((bits >> e) & 1u)) first = e;
  return first;
}

// the order that a selection ends in: one of the candidates, or (from == nullptr) the original
__global__ __launch_bounds__(256) void emit_order_kernel(const int32_t* __restrict__ from, int32_t* __restrict__ to, int K) {
  int i = blockIdx.x * 256 + threadIdx.x;
  if (i < K) to[i] = from ? from[i] : i;
}

// NVFP4 tensor scale of a launch: a host value, or a device float read by the kernel (dev != nullptr)
struct ScaleArg {
  float value;
  const float* dev;
};

// up to kMaxMomentBatches tensors of equal shape handled by one launch
struct TensorList {
  const uint16_t* p[kMaxMomentBatches];
};

// fewest rows a workgroup of the error evaluation covers (bounds the number of partial sums)
constexpr int kQeMinRowsPerBlock = 8;
constexpr int kQeMaxWaves = 16;           // waves of such a workgroup
constexpr size_t kQeLds = 150 * 1024;     // LDS its resident rows may take
constexpr int64_t kQeParts(int64_t rows) { return (rows / kQeMinRowsPerBlock + 1) * kQeMaxWaves; }

// A sum with what its additions lost (Knuth's two-sum): the errors of NVFP4 are differences of sums some hundred times as
// large, so a rounding of those is some hundred roundings of the error.
struct Sum2 {
  double s = 0.0, lost = 0.0;
  __device__ __forceinline__ void add(double x) {
    const double t = s + x, v = t - s;
    lost += (s - (t - v)) + (x - v);
    s = t;
  }
  __device__ __forceinline__ double value() const { return s + lost; }
};

// How the resident rows lie in LDS, as fp32 or as the bf16 values they are (packed: two instructions more for a pair of
// gathered values), for the widths that LDS holds them at.  fetch_ahead: staging chunks (8 channels x the rows) a thread has
// on their way.
struct QeWide4 { static constexpr int rows = 4, channel_bytes = 16, max_waves = 16, fetch_ahead = 1; };
struct QeWide2 { static constexpr int rows = 2, channel_bytes = 8, max_waves = 16, fetch_ahead = 2; };
struct QePacked4 { static constexpr int rows = 4, channel_bytes = 8, max_waves = 12, fetch_ahead = 2; };
struct QePacked2 { static constexpr int rows = 2, channel_bytes = 4, max_waves = 16, fetch_ahead = 3; };
enum QeRows : int { kQeWide4, kQeWide2, kQePacked4, kQePacked2 };

// channels of one work item of a lane: a whole NVFP4 group (its scale then needs no lane exchange and is
// worked out once), eight for the integer formats, whose groups span lanes
template <int FMT>
struct QeChunk { static constexpr int value = FMT == kNvfp4 ? 16 : 8; };

// (channel e's slot in the LDS image of the resident rows is slot e + e / 8: the spare slot per eight channels spreads the
// staging writes over the banks)

// Block scales of R rows' NVFP4 groups for the error: the decoded scale, and a reciprocal of it times T that is the
// quantizer's wherever the scale is not zero (a group whose scale is zero has error sum v^2 whatever its codes are, but its codes
// have to be finite).  Returns the largest amax / T, which says whether a scale saturated.
template <int R>
__device__ __forceinline__ float nv4_error_scales(const float (&amax)[R], float T, float encT, float (&inv)[R],
                                                  float (&value)[R]) {
  float u[R], t[R], largest = 0.0f;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    u[r] = amax[r] * encT;
    t[r] = div_const(u[r], 6.0f, 1.0f / 6.0f);
    largest = fmaxf(largest, u[r]);
  }
  uint32_t bytes;
#pragma unroll
  for (int r = 0; r < R; r += 2) e4m3_round2(t[r], t[r + 1], bytes, value[r], value[r + 1]);
  if (__builtin_expect(nv4_tensor_scale_is_tame(T), 1)) {        // uniform
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const float d = fmaxf(value[r], 0.001953125f) * T;         // 2^-9: the smallest scale
      const float q = __builtin_amdgcn_rcpf(d);
      inv[r] = __builtin_fmaf(__builtin_fmaf(-d, q, 1.0f), q, q);
    }
  } else {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const float d = value[r] * T;
      const bool normal = is_normal32(d);
      const float exact = recip_exact(d, normal);
      inv[r] = normal ? exact : 0.0f;
    }
  }
  return largest;
}

// Workgroup (x, y) evaluates rows [x * rows_per_block, (x + 1) * rows_per_block) of tensor y of
// the list (equal shapes) for every candidate order.  R rows at a time are staged in LDS (as ROWS says),
// channel-major with the R rows of a channel adjacent; the rows after them are already on
// their way from memory into registers while the resident ones are evaluated.  A candidate order
// comes as the byte offsets of its channels' slots (offs[cand][position]), so a lane reads the
// offsets of its chunk and gathers the R rows of each channel with one LDS read, no address
// arithmetic; the quantizer is the lane-cooperative one of the runtime kernels.  Integer formats: the
// error v - s t of an element is exact in fp32 and its square is accumulated in fp64.  NVFP4: the squared
// error of a group is sum v^2 - 2 d A + d^2 B (A = sum v q, B = sum q^2, d the group's scale): A and B are
// exact fp32 sums, the rest is fp64, and sum v^2 -- the same for every order -- is taken once when the rows
// are staged; the difference loses the bits by which sum v^2 exceeds the error (two decimal digits of
// fp64's sixteen for data that fill the format; an absolute 1e-15 of sum v^2 at worst).  Every wave owns a fixed run of work
// items (candidate, block of 64 chunks), candidate-major, sums a candidate's errors per lane and
// reduces them over the wave once per candidate and set of resident rows.  Lane c of every wave
// ends up with the wave's total for candidate c: part[y][c][x * waves + wave] (candidate-major, so
// that the sums over the workgroups read contiguous memory).
//
// Bound by the vector unit: for an element and order NVFP4 needs 16.7 cycles of a SIMD (two multiply-adds 5.7, its half of a
// conversion to E2M1 4.1 and back 2.1, the multiplication by the reciprocal 2.6, its half of a maximum 2.1), INT4 20.7 (the
// conversion to fp64 and the fma there 8.9), the rest is a group's scale and the work item's own, 222 instructions in all for 32
// elements.  8 x 4608 + 3072 rows of 12288, NVFP4, the whole selection 974 -> 880 us: rows asked for after the first
// item's offsets and not before them, the offsets of a set's first item kept ready, no LDS round trips where a candidate ends,
// block scales rounded two at a time on the conversion unit, the group's sum one fma chain (243 -> 222 instructions).
template <int FMT, int G, class ROWS>
__global__ __launch_bounds__(64 * ROWS::max_waves) void quant_error_kernel(TensorList xs, int rows, int K,
                                                          const int32_t* __restrict__ offs,
                                                          int n_cand, int identity_first, ScaleArg t_arg,
                                                          int rows_per_block, const uint32_t* __restrict__ differs,
                                                          double* __restrict__ part) {
  constexpr int R = ROWS::rows, SLOT = ROWS::channel_bytes;
  constexpr bool PACKED = SLOT == R * 2;
  typedef uint32_t vec_t __attribute__((ext_vector_type(SLOT / 4)));
  constexpr int C = QeChunk<FMT>::value;
  constexpr int PF = ROWS::fetch_ahead;
  constexpr bool kOffsetsAhead = SLOT < 16;  // the next item's offsets are loaded during the current item
  extern __shared__ __attribute__((aligned(16))) unsigned char slots[];      // (K + K / 8) * SLOT bytes
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int lane = tid & 63, n_waves = nthr >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint16_t* x = xs.p[blockIdx.y];
  const int row0 = blockIdx.x * rows_per_block;
  const int row_end = min(rows, row0 + rows_per_block);
  const int chunks8 = K / 8;               // staging granularity: one 16-byte load
  const int chunks = K / C;
  const int wave_chunks = (chunks + 63) >> 6;
  // Candidates that repeat an earlier order are left out.  Lane c works out whether candidate c does (one
  // load); the answer is used after the first rows have been requested (see below).
  int same_as_lane = lane;
  if (differs && lane < n_cand) same_as_lane = first_same_order(differs, lane);
  const float T = t_arg.dev ? *t_arg.dev : t_arg.value;           // uniform
  const float encT = (FMT == kNvfp4) ? nv4_enc_scale(T) : 0.0f;
  const double half_T = 0.5 * (double)T;
  // The offsets are used as LDS addresses as they are: the staged rows are the kernel's only LDS object and
  // start at address 0 (adding a base would cost one instruction per gathered channel).  Should a
  // toolchain ever place them elsewhere, every partial sum of the launch is made a NaN.
  typedef const __attribute__((address_space(3))) vec_t* lds_vec_ptr;
  const bool lds_at_zero = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)slots == 0u;

  // The rows of the workgroup as a buffer (at most 64 rows of 34128 channels): a read past its end gives zero without a
  // branch, so rows past the last count as zero rows, with error 0, and one offset is all an access needs.  A lane past the
  // row's last chunk reads what lies there and leaves it unused.
  const uint32_t row_bytes = (uint32_t)K * 2u;
  const auto rows_buf = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(x + (int64_t)row0 * K), 0, row_end > row0 ? (int)((uint32_t)(row_end - row0) * row_bytes) : 0, 0x00027000);
  auto fetch_row = [&](uint32_t row_at, int c) {         // row_at: byte offset of the row
    return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rows_buf, (int)(row_at + (uint32_t)c * 16u), 0, 0));
  };
  double v_sq = 0.0;                       // NVFP4: this thread's share of the sum of squares of the rows
  auto put = [&](int c, const uint4 (&p)[R]) {
    uint32_t w[R][4];
#pragma unroll
    for (int rr = 0; rr < R; ++rr) {
      w[rr][0] = p[rr].x; w[rr][1] = p[rr].y; w[rr][2] = p[rr].z; w[rr][3] = p[rr].w;
      if constexpr (FMT == kNvfp4) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const double lo = (double)bf16_lo(w[rr][j]), hi = (double)bf16_hi(w[rr][j]);
          v_sq = fma(lo, lo, v_sq);
          v_sq = fma(hi, hi, v_sq);
        }
      }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      vec_t o;
#pragma unroll
      for (int i = 0; i < SLOT / 4; ++i) {
        if constexpr (PACKED) {            // rows 2 i and 2 i + 1
          o[i] = __builtin_amdgcn_perm(w[2 * i + 1][j / 2], w[2 * i][j / 2], j & 1 ? 0x07060302u : 0x05040100u);
        } else {
          o[i] = j & 1 ? w[i][j / 2] & 0xFFFF0000u : w[i][j / 2] << 16;
        }
      }
      *reinterpret_cast<vec_t*>(slots + (size_t)(9 * c + j) * SLOT) = o;
    }
  };
  uint4 ahead[PF][R];
  auto fetch_ahead = [&](uint32_t at) {
#pragma unroll
    for (int f = 0; f < PF; ++f)
#pragma unroll
      for (int rr = 0; rr < R; ++rr) ahead[f][rr] = fetch_row(at + (uint32_t)rr * row_bytes, tid + f * nthr);
  };

  // the slot offsets of the C channels of work item (cand, blk) of this lane
  auto load_offsets = [&](int cand, int blk, int (&o)[C]) {
    const int c_lane = blk * 64 + lane;
    const int c = c_lane < chunks ? c_lane : 0;
    if (!(identity_first && cand == 0)) {
      const char* po = reinterpret_cast<const char*>(offs + (int64_t)(cand - identity_first) * K);
#pragma unroll
      for (int j = 0; j < C; j += 4) {
        const int4 q = *reinterpret_cast<const int4*>(po + ((uint32_t)c * (C * 4u) + j * 4u));
        o[j] = q.x; o[j + 1] = q.y; o[j + 2] = q.z; o[j + 3] = q.w;
      }
    } else {
      const int base = c * (C / 8 * 9) * SLOT;
#pragma unroll
      for (int j = 0; j < C; ++j) o[j] = base + ((j / 8) * 9 + (j & 7)) * SLOT;
    }
  };

  Sum2 acc;
  fetch_ahead(0u);
  // the orders to evaluate, four bits each (at most 16 candidates); the work items run over that list
  unsigned long long order_list = 0;
  int n_orders = 0;
  {
    const unsigned long long keep = __ballot(lane < n_cand && same_as_lane == lane);     // uniform
    for (int c = 0; c < n_cand; ++c) {
      if (!((keep >> c) & 1ull)) continue;
      order_list |= (unsigned long long)c << (4 * n_orders);
      ++n_orders;
    }
  }
  const int n_items = n_orders * wave_chunks;
  // The runs differ by one item; a SIMD's waves (w, w + 4, ...; a launch has a multiple of four) take neighbouring
  // runs, so that the SIMDs get the same number of items but for one.
  const int run = (wave & 3) * (n_waves >> 2) + (wave >> 2);
  const int it0 = run * n_items / n_waves, it1 = (run + 1) * n_items / n_waves;
  const int ord0 = it0 / wave_chunks, blk0 = it0 - ord0 * wave_chunks;       // uniform over the wave
  auto cand_of = [&](int ord) { return (int)((order_list >> (4 * ord)) & 15u); };
  uint32_t rg_at = 0;                      // byte offset of row rg
  int o_ahead[kOffsetsAhead ? C : 1];
  if constexpr (kOffsetsAhead) {
    if (it0 < it1) load_offsets(cand_of(ord0), blk0, o_ahead);
  }
  for (int rg = row0; rg < row_end; rg += R, rg_at += R * row_bytes) {
    __syncthreads();                       // the previous rows have been read by every wave
#pragma unroll
    for (int f = 0; f < PF; ++f) {
      const int c = tid + f * nthr;
      if (c < chunks8) put(c, ahead[f]);
    }
    for (int c = tid + PF * nthr; c < chunks8; c += nthr) {     // wider rows than the registers hold ahead
      uint4 p[R];
#pragma unroll
      for (int rr = 0; rr < R; ++rr) p[rr] = fetch_row(rg_at + (uint32_t)rr * row_bytes, c);
      put(c, p);
    }
    __syncthreads();
    // Loads return in issue order and a wave waits for all of them where the loop closes, so the order below matters: the
    // next set of rows is asked for inside the first item, once the offsets that it needs are there, and has that item's
    // time to arrive.  (Asked for before the first item they held its offsets up for a whole memory latency in every
    // set.)  The offsets of every later item are on their way while the item before it is evaluated, or asked for at
    // its start when four rows are resident: the registers do not hold both then, and a second workgroup of the compute unit
    // covers the wait.
    int ord = ord0, blk = blk0;
    int cand = cand_of(ord);
    if (it0 == it1) fetch_ahead(rg_at + R * row_bytes);           // no item of its own (uniform)
    double run = 0.0;                      // this lane's error of the current candidate
#pragma unroll 1                            // a first item of its own (peeled off) would cost registers
    for (int it = it0; it < it1; ++it) {
      // every lane runs the group reduction; a lane past the last chunk (its whole group is, K being a
      // multiple of the group size) works on chunk 0 and its result is dropped
      const bool live = blk * 64 + lane < chunks;
      int o[C];
      if constexpr (kOffsetsAhead) {
#pragma unroll
        for (int j = 0; j < C; ++j) o[j] = o_ahead[j];
      } else {
        load_offsets(cand, blk, o);
      }
      float v[R][C];
#pragma unroll
      for (int j = 0; j < C; ++j) {
        const vec_t g = *(lds_vec_ptr)(uintptr_t)(uint32_t)o[j];
#pragma unroll
        for (int rr = 0; rr < R; ++rr) v[rr][j] = !PACKED ? as_f32(g[rr]) : rr & 1 ? bf16_hi(g[rr / 2]) : bf16_lo(g[rr / 2]);
      }
      const bool cand_done = blk + 1 == wave_chunks || it + 1 == it1;     // uniform
      if constexpr (kOffsetsAhead) {
        const bool last = it + 1 == it1;             // then the first item's again, for the next set of rows
        load_offsets(last ? cand_of(ord0) : cand_done ? cand_of(ord + 1) : cand, last ? blk0 : cand_done ? 0 : blk + 1, o_ahead);
      }
      if (it == it0) {                                // uniform
        uint32_t next = rg_at + R * row_bytes;
        asm("" : "+s"(next));                         // the addresses are worked out here, not kept across the loop
        fetch_ahead(next);
      }
      constexpr bool kRows4 = FMT != kNvfp4 && R == 4 && G >= 32;    // scales shared out over a quad
      float amax[R];
#pragma unroll
      for (int rr = 0; rr < R; ++rr) {
        float a = 0.0f;
#pragma unroll
        for (int j = 0; j < C; ++j) a = fmaxf(a, fabsf(v[rr][j]));
        amax[rr] = kRows4 ? a : group_max<G / C>(a);
      }
      if constexpr (FMT == kNvfp4) {
        // A group's error is sum (v - q d)^2 = sum v^2 - 2 d A + d^2 B with A = sum v q and B = sum q^2
        // (q = +-E2M1 value, d = block scale x tensor scale).  sum v^2 does not depend on the order: it is
        // added once per row (v_sq below); the lane accumulates A and B in fp32, which is exact: an element
        // with q != 0 has |v| > d / 4, so every product v q is a multiple of U > d 2^-11 (bf16 v, q a
        // multiple of 1/2), and |A| <= 16 * 6 * amax < 2^24 U as long as amax <= 48 d -- true unless the block
        // scale saturated far beyond its largest value (a tensor scale much too small for the data: the
        // wave then takes the element-wise fp64 sum instead).  B <= 16 * 36 in steps of 1/4.
        // With d = b T (b the decoded block scale) the error is 2 T b ((T / 2) (b B) - A): b B is exact in fp32 (4 + 12
        // bits), (T / 2) (b B) in fp64, and the factor 2 T is applied to the sum of all groups at the end.
        float inv[R], value[R];
        const float largest = nv4_error_scales<R>(amax, T, encT, inv, value);
        const bool exact_sums = !__any(largest > 6.0f * 448.0f * 7.0f);          // uniform
        // eight elements on the conversion unit (a byte of `codes` per pair), decoded again
        auto quantize8 = [&](const float* x, float inv, float (&q)[8]) {
          uint32_t codes = 0u;
          codes = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(codes, x[0] * inv, x[1] * inv, 1.0f, 0);
          codes = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(codes, x[2] * inv, x[3] * inv, 1.0f, 1);
          codes = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(codes, x[4] * inv, x[5] * inv, 1.0f, 2);
          codes = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(codes, x[6] * inv, x[7] * inv, 1.0f, 3);
          const auto q0 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(codes, 1.0f, 0);
          const auto q1 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(codes, 1.0f, 1);
          const auto q2 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(codes, 1.0f, 2);
          const auto q3 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(codes, 1.0f, 3);
          q[0] = q0[0]; q[1] = q0[1]; q[2] = q1[0]; q[3] = q1[1];
          q[4] = q2[0]; q[5] = q2[1]; q[6] = q3[0]; q[7] = q3[1];
        };
        if (__builtin_expect(exact_sums, 1)) {
#pragma unroll
          for (int rr = 0; rr < R; ++rr) {
            float A = 0.0f, B = 0.0f;
#pragma unroll
            for (int j = 0; j < C; j += 8) {
              float q[8];
              quantize8(&v[rr][j], inv[rr], q);
#pragma unroll
              for (int u = 0; u < 8; ++u) {
                A = __builtin_fmaf(v[rr][j + u], q[u], A);
                B = __builtin_fmaf(q[u], q[u], B);
              }
            }
            const float b = live ? value[rr] : 0.0f;
            run = fma((double)b, fma(half_T, (double)(b * B), -(double)A), run);
          }
        } else {
          double far = 0.0;
#pragma unroll
          for (int rr = 0; rr < R; ++rr) {
            const double d = (double)value[rr] * (double)T;
#pragma unroll
            for (int j = 0; j < C; j += 8) {
              float q[8];
              quantize8(&v[rr][j], inv[rr], q);
#pragma unroll
              for (int u = 0; u < 8; ++u) {
                const double x = (double)v[rr][j + u];
                const double e = fma(-(double)q[u], d, x);      // product exact: 2 + 28 bits
                far = fma(e, e, far);
                far = fma(-x, x, far);                          // the part counted by v_sq
              }
            }
          }
          run += live ? far / (2.0 * (double)T) : 0.0;          // the factor of the other sums (T > 0: something saturated)
        }
      } else {
        IntScale s[R];
        if constexpr (kRows4) int_scales_rows4<FMT, G / C>(amax, lane, s);
        else int_scales<FMT, R>(amax, s);
        double errs[R];                             // one chain per resident row
#pragma unroll
        for (int rr = 0; rr < R; ++rr) errs[rr] = 0.0;
#pragma unroll
        for (int rr = 0; rr < R; ++rr) {
#pragma unroll
          for (int j = 0; j < C; ++j) {
            // The clip of the quantizer cannot act here: amax is the true maximum of the group, so
            // |x * inv| <= Q (1 + 3 * 2^-24) < Q + 1/2 and the rounding already lands on +-Q
            // (inv = 0 gives 0).  v_rndne_f32 rounds to the nearest integer, ties to even.
            const float t = __builtin_rintf(v[rr][j] * s[rr].inv);
            // v - s t is exact in binary32: for t != 0 both terms are multiples of the last place
            // of s and the difference is at most about s / 2, so it needs no more than 24 bits;
            // the fused multiply-add returns it unrounded
            const float e32 = __builtin_fmaf(-s[rr].s, t, v[rr][j]);
            const double e = (double)e32;
            errs[rr] = fma(e, e, errs[rr]);
          }
        }
        double err = errs[0];
#pragma unroll
        for (int rr = 1; rr < R; ++rr) err += errs[rr];
        run += live ? err : 0.0;
      }
      ++blk;
      if (cand_done) {                               // the candidate's last item of this wave
        const double total = wave_sum(run);          // fixed order
        acc.add(lane == cand ? total : 0.0);
        run = 0.0;
        blk = 0;
        ++ord;
        cand = cand_of(ord);
      }
    }
  }
  double err = acc.value();
  if constexpr (FMT == kNvfp4) {
    // every candidate's error contains the rows' sum of squares: the wave's share goes to each
    err = fma(2.0 * (double)T, acc.s, wave_sum(v_sq)) + 2.0 * (double)T * acc.lost;
  }
  if (!lds_at_zero) err = __builtin_nan("");
  if (lane < n_cand)
    part[((int64_t)blockIdx.y * n_cand + lane) * ((int64_t)gridDim.x * n_waves) + (int64_t)blockIdx.x * n_waves + wave] = err;
}

// offs[i] = byte offset of channel perm[i]'s slot for R resident rows (the error evaluation of one given order)
__global__ __launch_bounds__(256) void perm_to_offsets_kernel(const int32_t* __restrict__ perm, int K, int slot_bytes,
                                                              int32_t* __restrict__ offs) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= K) return;
  const int e = perm[i];
  offs[i] = (e + (e >> 3)) * slot_bytes;
}

// out[seg][c] = sum over the rows of segment seg of row_err[r][c]; one workgroup per
// (candidate, segment), fixed order.  Segments are consecutive runs of seg_rows rows.  not_below_zero: a
// sum that comes out negative (NVFP4's error of data the format holds exactly is zero up to the rounding
// of a difference) is returned as zero.
__global__ __launch_bounds__(256) void reduce_rows_kernel(const double* __restrict__ row_err,
                                                          int64_t seg_rows, int n_cand, int out_stride,
                                                          int not_below_zero, double* __restrict__ out) {
  __shared__ double red[256];
  const int c = blockIdx.x;
  const double* base = row_err + (int64_t)blockIdx.y * seg_rows * n_cand;
  double s = 0.0;
  for (int64_t r = threadIdx.x; r < seg_rows; r += 256) s += base[r * n_cand + c];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[(int64_t)blockIdx.y * out_stride + c] = not_below_zero && red[0] < 0.0 ? 0.0 : red[0];
}

// Everything the host needs for the decision, in one launch.  Workgroup b of the grid computes
// one fixed-order sum (per-thread strided partial sums, then a binary tree) into out[]:
//   b <  n_cand * n_batches         error of candidate b % n_cand on calibration batch b / n_cand
//                                   -> out[batch * kMaxCand + cand]
//   next n_cand                     error of the candidate on the weights -> out[n_batches * kMaxCand + cand]
//   next 2                          sum of act_sumsq, sum of w_sumsq      -> out[(n_batches + 1) * kMaxCand + 0 / 1]
//   next n_alpha                    number of channels candidate j moves  -> out[... + 2 + j] (as a double)
struct TailArgs {
  const double* x_part;     // [n_batches][n_cand][x_parts]
  const double* w_part;     // [n_cand][w_parts]
  const double* act_sumsq;
  const double* w_sumsq;
  const int32_t* cands;     // [n_alpha][K]
  const uint32_t* differs;  // per alpha: which earlier candidates differ; a repeated order takes the first one's sums
  int64_t x_parts, w_parts, K;
  int n_cand, n_batches, n_alpha;
};

// s + p[i0] + p[i0 + stride] + ... (i < n), in that order, with eight loads in flight at a time (a plain
// loop waits out one memory latency per element)
__device__ __forceinline__ double strided_sum(const double* __restrict__ p, int64_t i0, int64_t n, int64_t stride) {
  double s = 0.0;
  int64_t i = i0;
  for (; i + 7 * stride < n; i += 8 * stride) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = p[i + u * stride];
#pragma unroll
    for (int u = 0; u < 8; ++u) s += v[u];
  }
  for (; i < n; i += stride) s += p[i];
  return s;
}

__global__ __launch_bounds__(256) void select_tail_kernel(TailArgs a, double* __restrict__ out) {
  __shared__ double red[256], red_lost[256];
  const int n_x = a.n_cand * a.n_batches;
  int b = blockIdx.x;
  double s = 0.0, lost = 0.0;
  int64_t dst;
  if (b < n_x + a.n_cand) {
    const bool is_w = b >= n_x;
    const int seg = is_w ? 0 : b / a.n_cand, c = is_w ? b - n_x : b % a.n_cand;
    const int64_t n = is_w ? a.w_parts : a.x_parts;
    const double* base = is_w ? a.w_part : a.x_part + (int64_t)seg * n * a.n_cand;
    const double* p = base + (int64_t)first_same_order(a.differs, c) * n;
    Sum2 sum;
    int64_t i = threadIdx.x;
    for (; i + 7 * 256 < n; i += 8 * 256) {
      double v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = p[i + u * 256];
#pragma unroll
      for (int u = 0; u < 8; ++u) sum.add(v[u]);
    }
    for (; i < n; i += 256) sum.add(p[i]);
    s = sum.s;
    lost = sum.lost;
    dst = (int64_t)(is_w ? a.n_batches : seg) * kMaxCand + c;
  } else if (b < n_x + a.n_cand + 2) {
    const int which = b - n_x - a.n_cand;
    const double* p = which ? a.w_sumsq : a.act_sumsq;
    s = strided_sum(p, threadIdx.x, a.K, 256);
    dst = (int64_t)(a.n_batches + 1) * kMaxCand + which;
  } else {
    const int j = b - n_x - a.n_cand - 2;
    const int32_t* p = a.cands + (int64_t)j * a.K;
    int n = 0;
    int64_t i = threadIdx.x;
    for (; i + 7 * 256 < a.K; i += 8 * 256) {
      int32_t v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = p[i + u * 256];
#pragma unroll
      for (int u = 0; u < 8; ++u) n += (v[u] != (int32_t)(i + u * 256));
    }
    for (; i < a.K; i += 256) n += (p[i] != (int32_t)i);
    s = (double)n;                                    // small integers: every sum below is exact
    dst = (int64_t)(a.n_batches + 1) * kMaxCand + 2 + j;
  }
  Sum2 sum{s, lost};
  red[threadIdx.x] = s;
  red_lost[threadIdx.x] = lost;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st) {
      sum.add(red[threadIdx.x + st]);
      sum.lost += red_lost[threadIdx.x + st];
      red[threadIdx.x] = sum.s;
      red_lost[threadIdx.x] = sum.lost;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) out[dst] = sum.value();
}

// Launch shape of the error evaluation of n_cand orders for `rows` rows per tensor of width K; most_rows: those of the tensor
// of the call that has most.
struct QeShape {
  QeRows kind;
  int r;                 // rows resident in LDS together (2 or 4)
  int slot;              // bytes of a channel there
  int threads;
  int rows_per_block;
  int blocks;            // per tensor
  size_t shmem;
  int parts() const { return blocks * (threads / 64); }    // partial sums per tensor and candidate
};

static QeShape qe_shape(pq_format fmt, int group, int64_t rows, int64_t K, int n_tensors, int n_cand, int64_t most_rows) {
  QeShape q;
  const bool nv = fmt == PQ_FMT_NVFP4;
  const int chunk = nv ? QeChunk<kNvfp4>::value : QeChunk<kInt4>::value;
  const size_t slots = (size_t)(K + K / 8);
  // Resident rows: four where LDS holds them, one gather and one load of offsets then serve four elements.  As fp32 up to K =
  // 8533, also where that leaves room for one workgroup a unit only (K above 4551): against two rows a whole selection takes
  // 0.86 to 0.99 of the time over K = 4096 to 8448.  Wider rows up to K = 17066: the integer formats as bf16 (against two
  // rows of fp32: INT4 g64 1024 + 1024 + 1024 rows of 12288 160 -> 151 us, g32 2 x 1500 + 2000 of 16384 228 -> 216), which share
  // a group's scale arithmetic over four rows; NVFP4, which does not, two rows of fp32 (2 x 1500 + 2000 of 16384 210
  // against 218, 3 x 4608 + 3072 of 10240 357 against 366, 8 x 4608 + 3072 of 12288 883 against 874).  Wider still two rows of
  // bf16 instead of one of fp32: INT4 g256 512 + 512 of 20480 290 -> 256, NVFP4 1500 + 2000 of 32768 380 -> 364.  So where the
  // call's tensors have no more than two rows, half of four would be zeros: INT4 g256 2 x 15616 11.2 -> 9.3 us.
  q.kind = slots * QeWide4::channel_bytes <= kQeLds                     ? kQeWide4
           : slots * QeWide2::channel_bytes <= kQeLds && nv             ? kQeWide2
           : slots * QeWide2::channel_bytes <= kQeLds && most_rows > 2  ? kQePacked4
                                                                        : kQePacked2;
  q.r = q.kind == kQeWide4 || q.kind == kQePacked4 ? 4 : 2;
  q.slot = q.kind == kQeWide4 ? QeWide4::channel_bytes : q.kind == kQePacked2 ? QePacked2::channel_bytes : QeWide2::channel_bytes;
  q.shmem = slots * q.slot;
  // Waves, a multiple of four: the waves of a workgroup are dealt to the four SIMDs in turn, both workgroups of a
  // unit from the same SIMD on, and the busiest SIMD sets the pace (INT4, K = 3072: 315 us with nine waves, 254 with
  // eight, 246 with twelve; NVFP4, K = 12288, two batches: 403 with fourteen, 389 with sixteen).  Two workgroups share
  // a unit where their rows fit its LDS twice (one stages while the other computes): half of the waves that the
  // registers allow each (the NVFP4 instances need up to 128 a lane: sixteen waves a unit; the integer ones up to 80:
  // twenty-four), sixteen otherwise.  No more waves than there are work items (candidate x block of 64 chunks), rounded up to four.
  const int items = n_cand * (int)((K / chunk + 63) / 64);
  const bool two = 2 * q.shmem <= 160 * 1024 && q.kind != kQePacked4;
  const int max_waves = q.kind == kQePacked4 ? QePacked4::max_waves : two ? (nv ? 8 : 12) : kQeMaxWaves;
  q.threads = 64 * (items < max_waves ? (items + 3) / 4 * 4 : max_waves);
  // Rows per workgroup: the workgroups run in rounds of as many as the chip holds at once (256 compute
  // units, one or two each), every round lasts about as long as a workgroup's rows plus a fixed start-up
  // (taken as half a row); among kQeMinRowsPerBlock .. 64 rows take the smallest size whose total is
  // within 2 % of the shortest (smaller workgroups even out better when their times differ).
  const int64_t resident = (two ? 2 : 1) * 256;
  const int64_t lo = (kQeMinRowsPerBlock + q.r - 1) / q.r * q.r;
  auto cost_of = [&](int64_t rpb) {
    const int64_t wgs = (rows + rpb - 1) / rpb * n_tensors;
    return (double)((wgs + resident - 1) / resident) * ((double)rpb + 0.5);
  };
  double best_cost = cost_of(lo);
  for (int64_t rpb = lo; rpb <= 64; rpb += q.r) best_cost = cost_of(rpb) < best_cost ? cost_of(rpb) : best_cost;
  int64_t best_rpb = lo;
  while (cost_of(best_rpb) > 1.02 * best_cost) best_rpb += q.r;
  q.rows_per_block = (int)best_rpb;
  q.blocks = (int)((rows + best_rpb - 1) / best_rpb);
  return q;
}

template <int FMT, int G, class ROWS>
static int launch_qe_r(const TensorList& xs, int n_tensors, int64_t rows, int K, const QeShape& q,
                       const int32_t* offs, int n_cand, int identity_first, ScaleArg T, const uint32_t* same_as,
                       double* part, hipStream_t st) {
  auto kern = quant_error_kernel<FMT, G, ROWS>;
  static std::atomic<uint64_t> raised{0};              // to the most any launch of the instance may ask for
  if (q.shmem > 48 * 1024) {
    if (int rc = allow_lds(reinterpret_cast<const void*>(kern), kQeLds, raised, "hipFuncSetAttribute(quant_error_kernel)"))
      return rc;
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)q.blocks, (unsigned)n_tensors), dim3(q.threads), q.shmem, st, xs,
                     (int)rows, K, offs, n_cand, identity_first, T, q.rows_per_block, same_as, part);
  return check_hip(hipGetLastError(), "quant_error_kernel");
}

template <int FMT, int G>
static int launch_qe(const TensorList& xs, int n_tensors, int64_t rows, int K, const QeShape& q,
                     const int32_t* offs, int n_cand, int identity_first, ScaleArg T, const uint32_t* same_as,
                     double* part, hipStream_t st) {
#define PQ_ARGS (xs, n_tensors, rows, K, q, offs, n_cand, identity_first, T, same_as, part, st)
  if (q.kind == kQeWide4) return launch_qe_r<FMT, G, QeWide4> PQ_ARGS;
  if (q.kind == kQePacked2) return launch_qe_r<FMT, G, QePacked2> PQ_ARGS;
  return launch_qe_r<FMT, G, std::conditional_t<FMT == kNvfp4, QeWide2, QePacked4>> PQ_ARGS;
#undef PQ_ARGS
}

// part: [n_tensors][n_cand][q.parts()]; offs: the candidate orders as offsets of slots of q.slot bytes
static int launch_quant_error(pq_format fmt, int group, const TensorList& x, int n_tensors, int64_t rows,
                              int K, const QeShape& q, const int32_t* offs, int n_cand,
                              int identity_first, ScaleArg T, const uint32_t* same_as, double* part,
                              hipStream_t st) {
  if (rows > 0x7FFFFFFF) return fail(PQ_ERR_SHAPE, "too many rows");
  if (q.shmem > kQeLds) return fail(PQ_ERR_SHAPE, "K=%d too large for the LDS-resident row", K);   // the entry points refuse this earlier
  if (fmt == PQ_FMT_NVFP4)
    return launch_qe<kNvfp4, 16>(x, n_tensors, rows, K, q, offs, n_cand, identity_first, T, same_as, part, st);
#define PQ_INT_CASE(F, FE)                                                                                  \
  if (fmt == F) {                                                                                           \
    switch (group) {                                                                                        \
      case 32: return launch_qe<FE, 32>(x, n_tensors, rows, K, q, offs, n_cand, identity_first, T, same_as, part, st);   \
      case 64: return launch_qe<FE, 64>(x, n_tensors, rows, K, q, offs, n_cand, identity_first, T, same_as, part, st);   \
      case 128: return launch_qe<FE, 128>(x, n_tensors, rows, K, q, offs, n_cand, identity_first, T, same_as, part, st); \
      case 256: return launch_qe<FE, 256>(x, n_tensors, rows, K, q, offs, n_cand, identity_first, T, same_as, part, st); \
    }                                                                                                       \
  }
  PQ_INT_CASE(PQ_FMT_INT4, kInt4)
  PQ_INT_CASE(PQ_FMT_INT3, kInt3)
#undef PQ_INT_CASE
  return fail(PQ_ERR_FORMAT, "unsupported (format, group) = (%d, %d)", (int)fmt, group);
}

// ------------------------------------------------------------------------- workspace layout
struct SelectWs {
  double* keys;      // [PQ_MAX_ALPHAS][K]
  int32_t* cands;    // [PQ_MAX_ALPHAS][K]
  int32_t* rank;     // [PQ_MAX_ALPHAS][K] position of every channel in the sorted order
  int32_t* offs;     // [PQ_MAX_ALPHAS][K] the candidates as LDS slot offsets of the error evaluation
  uint32_t* same_as; // [PQ_MAX_ALPHAS] per alpha: a bit per earlier candidate whose order differs (rank_scatter_kernel)
  double* row_err;   // partial error sums: [n_batches][n_cand][parts(M)], then [n_cand][parts(N)]
  double* sums;      // [(n_batches + 1) * kMaxCand + 2 + PQ_MAX_ALPHAS]: per-batch errors, weight
                     // errors, |X|^2, |W|^2, moved-channel counts
};

static size_t carve_select(void* base, int64_t M, int64_t N, int64_t K, int n_batches, SelectWs* w) {
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off = align_up(off + bytes, 256);
    return o;
  };
  size_t o_keys = take((size_t)PQ_MAX_ALPHAS * K * 8);
  size_t o_cands = take((size_t)PQ_MAX_ALPHAS * K * 4);
  size_t o_rank = take((size_t)PQ_MAX_ALPHAS * K * 4);
  size_t o_offs = take((size_t)PQ_MAX_ALPHAS * K * 4);
  size_t o_same = take((size_t)kMaxCand * 4);
  // a workgroup covers at least kQeMinRowsPerBlock rows with at most kQeMaxWaves waves: no more
  // partial sums than kQeParts(rows) per tensor
  size_t o_rowerr = take((size_t)((int64_t)n_batches * kQeParts(M) + kQeParts(N)) * kMaxCand * 8);
  size_t o_sums = take(((size_t)(n_batches + 1) * kMaxCand + 2 + PQ_MAX_ALPHAS) * 8);
  if (w) {
    char* b = (char*)base;
    w->keys = (double*)(b + o_keys);
    w->cands = (int32_t*)(b + o_cands);
    w->rank = (int32_t*)(b + o_rank);
    w->offs = (int32_t*)(b + o_offs);
    w->same_as = (uint32_t*)(b + o_same);
    w->row_err = (double*)(b + o_rowerr);
    w->sums = (double*)(b + o_sums);
  }
  return off;
}

size_t select_workspace_bytes(int64_t M, int64_t N, int64_t K, int n_batches) {
  return carve_select(nullptr, M, N, K, n_batches, nullptr);
}

// partial sums, then the given order as slot offsets
size_t quant_error_workspace_bytes(int64_t rows, int64_t K) {
  return align_up((size_t)kQeParts(rows) * 8, 256) + align_up((size_t)K * 4, 256);
}

int run_quant_error(pq_format fmt, int group, const void* x, int64_t rows, int64_t K,
                    const int32_t* perm, float ts, double* err_out, void* ws, hipStream_t st) {
  double* part = (double*)ws;
  TensorList tl;
  for (int b = 0; b < kMaxMomentBatches; ++b) tl.p[b] = (const uint16_t*)x;
  const QeShape q = qe_shape(fmt, group, rows, K, 1, 1, rows);
  int32_t* offs = nullptr;
  if (perm) {
    offs = (int32_t*)((char*)ws + align_up((size_t)kQeParts(rows) * 8, 256));
    hipLaunchKernelGGL(perm_to_offsets_kernel, dim3((unsigned)((K + 255) / 256)), dim3(256), 0, st, perm, (int)K,
                       q.slot, offs);
  }
  int rc = launch_quant_error(fmt, group, tl, 1, rows, (int)K, q, offs, 1, perm ? 0 : 1, ScaleArg{ts, nullptr},
                              nullptr, part, st);
  if (rc) return rc;
  hipLaunchKernelGGL(reduce_rows_kernel, dim3(1, 1), dim3(256), 0, st, part, (int64_t)q.parts(), 1, 1,
                     fmt == PQ_FMT_NVFP4 ? 1 : 0, err_out);
  return check_hip(hipGetLastError(), "reduce_rows_kernel");
}

// rank[n][K] of the channels in n descending orders; order[n][K] is scratch (overwritten by the scatter that follows)
static void launch_ranks(const double* act_sumsq, const double* w_sumsq, int64_t K, const AlphaList& al, int n,
                         double* keys, int32_t* order, int32_t* rank, uint32_t* differs, hipStream_t st) {
  const unsigned kb = (unsigned)((K + kSortBlock - 1) / kSortBlock);
  hipLaunchKernelGGL(block_order_kernel, dim3(kb, n), dim3(kSortBlock * kSortShares), 0, st, act_sumsq, w_sumsq, K, al, keys, order,
                     rank, differs);
  hipLaunchKernelGGL(rank_merge_kernel, dim3(kb, (kb + kMergeBlocks - 1) / kMergeBlocks, n), dim3(kSortBlock), 0, st,
                     keys, order, (int)K, (int)kb, rank);
}

// The candidate orders of the alpha grid (joint score, descending stable sort) into
// cands[n_alpha][K]; keys [PQ_MAX_ALPHAS][K] doubles and rank [PQ_MAX_ALPHAS][K] ints are scratch.
// With offs ([n_alpha][K]), the same orders are also written as slot offsets of slot_bytes a slot.
int launch_candidate_orders(const double* act_sumsq, const double* w_sumsq, int64_t K, const double* alphas,
                            int n_alpha, double* keys, int32_t* rank, int32_t* cands, hipStream_t st,
                            int32_t* offs, int slot_bytes, uint32_t* differs) {
  const unsigned kb = (unsigned)((K + 255) / 256);
  AlphaList al;
  for (int j = 0; j < PQ_MAX_ALPHAS; ++j) al.a[j] = j < n_alpha ? alphas[j] : 0.0;
  launch_ranks(act_sumsq, w_sumsq, K, al, n_alpha, keys, cands, rank, differs, st);
  hipLaunchKernelGGL(rank_scatter_kernel, dim3(kb, n_alpha), dim3(256), 0, st, rank, (int)K, cands, offs,
                     slot_bytes, differs);
  return check_hip(hipGetLastError(), "key/rank kernels");
}

// ---- orders of the ablation (paper Tab. 2a) that are not a sort by a statistic
// round-robin: rank r of `order` goes to group r mod (K / g), slot r div (K / g)
__global__ __launch_bounds__(256) void round_robin_kernel(const int32_t* __restrict__ order, int K, int g,
                                                         int32_t* __restrict__ perm) {
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= K) return;
  const int n_groups = K / g;
  perm[(r % n_groups) * g + r / n_groups] = order[r];
}

// random: key[i] = -(splitmix64(seed + i) >> 11) as a double (53 bits: exact), so that the descending
// stable sort used for the scores gives ascending hashes with ties in ascending channel order
__global__ __launch_bounds__(256) void random_key_kernel(uint64_t seed, int K, double* __restrict__ keys) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= K) return;
  uint64_t z = seed + (uint64_t)i + 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z = z ^ (z >> 31);
  keys[i] = -(double)(z >> 11);
}

int launch_round_robin(const int32_t* order, int64_t K, int group, int32_t* perm, hipStream_t st) {
  hipLaunchKernelGGL(round_robin_kernel, dim3((unsigned)((K + 255) / 256)), dim3(256), 0, st, order, (int)K, group, perm);
  return check_hip(hipGetLastError(), "round_robin_kernel");
}

size_t random_order_workspace_bytes(int64_t K) { return align_up((size_t)K * 8, 256) + align_up((size_t)K * 4, 256); }

int launch_random_order(uint64_t seed, int64_t K, int32_t* perm, void* ws, hipStream_t st) {
  double* keys = (double*)ws;
  int32_t* rank = (int32_t*)((char*)ws + align_up((size_t)K * 8, 256));
  const unsigned kb = (unsigned)((K + 255) / 256);
  hipLaunchKernelGGL(random_key_kernel, dim3(kb), dim3(256), 0, st, seed, (int)K, keys);
  launch_ranks(nullptr, nullptr, K, AlphaList{}, 1, keys, perm, rank, nullptr, st);
  hipLaunchKernelGGL(rank_scatter_kernel, dim3(kb, 1), dim3(256), 0, st, rank, (int)K, perm,
                     (int32_t*)nullptr, 0, (uint32_t*)nullptr);
  return check_hip(hipGetLastError(), "random order kernels");
}

// from == nullptr: the original order.  A kernel, not a copy: the device waits for it, and a copy command takes the host
// longer to hand over than a launch
int launch_emit_order(const int32_t* from, int32_t* to, int64_t K, hipStream_t st) {
  hipLaunchKernelGGL(emit_order_kernel, dim3((unsigned)((K + 255) / 256)), dim3(256), 0, st, from, to, (int)K);
  return check_hip(hipGetLastError(), "emit_order_kernel");
}

// A pinned host buffer of at least n doubles that the calling thread keeps until it ends
// (a device-to-host copy into pageable memory goes through a staging copy and costs some 10 us
// more).  Grown, never shrunk; nullptr when the allocation fails.
struct PinnedBuffer {
  double* buf = nullptr;
  size_t cap = 0;
  ~PinnedBuffer() {                      // runs when the owning thread ends
    if (buf) (void)hipHostFree(buf);
  }
};
double* pinned_doubles(size_t n) {
  thread_local PinnedBuffer pb;
  if (n > pb.cap) {
    if (pb.buf) (void)hipHostFree(pb.buf);
    pb.buf = nullptr;
    pb.cap = 0;
    const size_t want = n < 512 ? 512 : n;
    void* p = nullptr;
    if (hipHostMalloc(&p, want * sizeof(double), hipHostMallocDefault) != hipSuccess) {
      (void)hipGetLastError();
      return nullptr;
    }
    pb.buf = (double*)p;
    pb.cap = want;
  }
  return pb.buf;
}

int run_select(pq_format fmt, int group, const double* act_sumsq, const double* w_sumsq, int64_t K,
               const void* const* x_calib, int n_batches, int64_t M, const void* w, int64_t N,
               float act_ts, float w_ts, const float* act_ts_dev, const float* w_ts_dev, const double* alphas,
               int n_alpha, double tau, int32_t* perm_out, pq_select_report* report, void* ws, hipStream_t st) {
  SelectWs W;
  carve_select(ws, M, N, K, n_batches, &W);
  const int n_cand = n_alpha + 1;            // candidate 0 is the original order
  int rc;
  // activations: all batches of a launch share one grid (up to kMaxMomentBatches per launch)
  const int64_t most_rows = M > N ? M : N;
  const QeShape qa = qe_shape(fmt, group, M, K, n_batches < kMaxMomentBatches ? n_batches : kMaxMomentBatches, n_cand,
                              most_rows);
  const QeShape qw = qe_shape(fmt, group, N, K, 1, n_cand, most_rows);       // the same resident rows: one set of offsets
  if ((rc = launch_candidate_orders(act_sumsq, w_sumsq, K, alphas, n_alpha, W.keys, W.rank, W.cands, st, W.offs,
                                    qa.slot, W.same_as)))
    return rc;
  double* sums = W.sums;
  for (int b0 = 0; b0 < n_batches; b0 += kMaxMomentBatches) {
    const int nb = n_batches - b0 < kMaxMomentBatches ? n_batches - b0 : kMaxMomentBatches;
    TensorList tl;
    for (int b = 0; b < kMaxMomentBatches; ++b) tl.p[b] = (const uint16_t*)x_calib[b0 + (b < nb ? b : 0)];
    rc = launch_quant_error(fmt, group, tl, nb, M, (int)K, qa, W.offs, n_cand, 1, ScaleArg{act_ts, act_ts_dev},
                            W.same_as, W.row_err + (size_t)b0 * qa.parts() * n_cand, st);
    if (rc) return rc;
  }
  double* w_part = W.row_err + (size_t)n_batches * qa.parts() * n_cand;
  TensorList wl;
  for (int b = 0; b < kMaxMomentBatches; ++b) wl.p[b] = (const uint16_t*)w;
  rc = launch_quant_error(fmt, group, wl, 1, N, (int)K, qw, W.offs, n_cand, 1, ScaleArg{w_ts, w_ts_dev}, W.same_as,
                          w_part, st);
  if (rc) return rc;
  TailArgs ta{W.row_err, w_part, act_sumsq, w_sumsq, W.cands, W.same_as, qa.parts(), qw.parts(), K, n_cand, n_batches,
              n_alpha};
  hipLaunchKernelGGL(select_tail_kernel, dim3((unsigned)(n_cand * (n_batches + 1) + 2 + n_alpha)), dim3(256), 0,
                     st, ta, sums);
  if ((rc = check_hip(hipGetLastError(), "select_tail_kernel"))) return rc;

  const size_t n_tot = (size_t)(n_batches + 1) * kMaxCand;      // offset of the two totals
  const size_t n_sums = n_tot + 2 + (size_t)n_alpha;
  double* h = pinned_doubles(n_sums);
  if (!h) return fail(PQ_ERR_HIP, "pq_select_perm: no pinned host memory for %zu sums", n_sums);
  if ((rc = check_hip(hipMemcpyAsync(h, sums, n_sums * 8, hipMemcpyDeviceToHost, st), "copy sums"))) return rc;
  if ((rc = check_hip(hipStreamSynchronize(st), "hipStreamSynchronize"))) return rc;

  const double sum_x2 = h[n_tot], sum_w2 = h[n_tot + 1];
  double E[kMaxCand];
  for (int c = 0; c < n_cand; ++c) {
    double ex = 0.0;
    for (int b = 0; b < n_batches; ++b) ex += h[(size_t)b * kMaxCand + c];
    double ew = h[(size_t)n_batches * kMaxCand + c];
    if (fmt == PQ_FMT_NVFP4) {
      // NVFP4 errors are differences known to about 1e-15 of the tensor's sum of squares: below 1e-13 of it
      // they are not told from zero (data the format holds exactly), and are reported as zero
      if (ex < 1e-13 * sum_x2) ex = 0.0;
      if (ew < 1e-13 * sum_w2) ew = 0.0;
    }
    E[c] = ex / sum_x2 + ew / sum_w2;
  }
  int best = 0;
  for (int j = 1; j < n_alpha; ++j)
    if (E[1 + j] < E[1 + best]) best = j;         // first minimum: smallest alpha on ties
  const double e_orig = E[0], e_best = E[1 + best];
  const bool accepted = h[n_tot + 2 + best] != 0.0 && e_orig > 0.0 && ((e_orig - e_best) / e_orig > tau);
  memset(report, 0, sizeof(*report));
  report->accepted = accepted ? 1 : 0;
  report->alpha_index = best;
  report->e_orig = e_orig;
  report->e_best = e_best;
  for (int j = 0; j < n_alpha; ++j) report->e_cand[j] = E[1 + j];
  report->sum_x2 = sum_x2;
  report->sum_w2 = sum_w2;
  return launch_emit_order(accepted ? W.cands + (int64_t)best * K : nullptr, perm_out, K, st);
}

}  // namespace pq
