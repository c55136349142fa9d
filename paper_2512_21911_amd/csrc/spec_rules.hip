// Expert skipping of the sparse mixture of experts (Sec. 3.5, Eq. 15-16) and acceptance /
// resampling of the draft tokens (Sec. 2.1, Eq. 2-3): small, latency-bound kernels.
//
//   moe kernels   sixteen lanes per token (32 for more than sixteen experts), lane j holds the
//                 weight of the token's j-th expert.  A lane's rank (weights below it, equal
//                 weights by position) comes from k broadcasts; the weights move to their rank's
//                 lane and every lane adds its prefix sequentially in ascending order (the order
//                 the sums are defined in).
//   median        one workgroup per skip size: 4-pass radix select over the tokens' ratios
//                 (positive floats order like their bit patterns), twice when T is even.
//   accept        one workgroup per sequence: the gamma acceptance tests in one wavefront, then,
//                 if a position was rejected, the residual mass of every chunk of 256 consecutive
//                 tokens (a wavefront reads a chunk as one contiguous kilobyte per distribution),
//                 a scan of the chunk sums, and a walk of the one chunk the target falls in.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "svf.h"
#include "svf_rules.h"

namespace {

// The kernel is a chain: launch, one round trip for weights and thresholds, some hundred dependent
// instructions.  Hence small workgroups, everything requested at once, loops of a length known at
// compile time, and broadcasts inside a row of sixteen lanes by an operand modifier (a shuffle is a
// trip through LDS).  256 tokens of 8, 16, 17, 32 experts: 2.3, 2.5, 2.8, 3.2 us a call (2.0 is an empty launch),
// against 2.7, 3.3, 3.4, 4.5 with 32 lanes per token, loops of run-time length, the sorted weights in LDS, and the
// thresholds loaded behind the sums; 65 536 tokens: 6.0, 6.6, 12.2, 16.3 against 8.8, 12.7, 13.2, 20.7 us (24.4 for 17
// and 32 experts with shuffles in loops of 32).
constexpr int kMoeThreads = 64;

// A value per lane of a token's 16 or 32 lanes, each of which can be had in all of them: 16 lanes are a row of the
// wavefront; of 32, both rows hold the first row's values and the second row's.
template <int LANES>
struct TokenLanes {
  float low, high;
  __device__ __forceinline__ explicit TokenLanes(float x) : low(x), high(x) {
    if constexpr (LANES == 32) {                         // (odd rows of the one against even rows of the other)
      const auto rows = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
      low = __uint_as_float(rows[0]);
      high = __uint_as_float(rows[1]);
    }
  }
  template <int L>
  __device__ __forceinline__ float lane() const {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(L < 16 ? low : high), 0x150 + (L & 15), 0xf, 0xf, true));   // row_newbcast
  }
};

// Weights of lanes 0 .. L that come before lane j's, w, in ascending order (equal weights: by position).
template <int LANES, int L>
__device__ __forceinline__ int rank_upto(const TokenLanes<LANES>& all, float w, int j) {
  const float o = all.template lane<L>();
  const int r = (o < w || (o == w && L < j)) ? 1 : 0;
  if constexpr (L > 0) return r + rank_upto<LANES, L - 1>(all, w, j);
  else return r;
}
// total: sorted[0] + ... + sorted[L], added in that order; prefix: lane j's sum up to its own.
template <int LANES, int L>
__device__ __forceinline__ void sums_upto(const TokenLanes<LANES>& sorted, int j, float& prefix, float& total) {
  if constexpr (L > 0) sums_upto<LANES, L - 1>(sorted, j, prefix, total);
  total += sorted.template lane<L>();
  if (L == j) prefix = total;
}

// Rank of lane j's weight among the token's k <= KMAX weights and the token's sorted prefix sums:
// prefix = sum of the weights of rank <= j.  Lanes j >= k take part with a weight that comes behind
// all others and count nothing in the sums (adding zero to them changes no bit).
template <int KMAX>
struct MoeToken {
  static constexpr int kLanes = KMAX <= 16 ? 16 : 32;
  static constexpr int kPerWorkgroup = kMoeThreads / kLanes;
  int rank;
  float prefix, total;
  __device__ __forceinline__ MoeToken(float w, int j, int k) {
    const float mine = j < k ? w : INFINITY;
    rank = rank_upto<kLanes, KMAX - 1>(TokenLanes<kLanes>(mine), mine, j);
    // (a lane past KMAX counts KMAX at most and writes behind the k lanes that are read)
    const int to = ((int)threadIdx.x & ~(kLanes - 1)) + (j < KMAX ? rank : j);
    float sorted = __int_as_float(__builtin_amdgcn_ds_permute(4 * to, __float_as_int(mine)));
    if (j >= k) sorted = 0.f;
    prefix = total = 0.f;
    sums_upto<kLanes, KMAX - 1>(TokenLanes<kLanes>(sorted), j, prefix, total);
  }
};

// grid: ceil(T / tokens per workgroup)
template <int KMAX>
__global__ __launch_bounds__(kMoeThreads) void moe_skip_kernel(const float* __restrict__ w, int T, int k, int m,
                                                               const float* __restrict__ beta, int32_t* n_skip,
                                                               uint32_t* keep_mask) {
  typedef MoeToken<KMAX> Token;
  const int j = threadIdx.x & (Token::kLanes - 1), tl = threadIdx.x / Token::kLanes;
  const int t = blockIdx.x * Token::kPerWorkgroup + tl;
  const bool live = t < T;
  // (both requested before either is waited for, from addresses that are valid in every lane)
  const float wj = w[(int64_t)min(t, T - 1) * k + min(j, k - 1)];
  const float bj = beta[min(j, m - 1)];
  const Token tok(wj, j, k);
  // lane j looks at skip size i = j + 1
  const bool ok = live && j < m && tok.prefix / tok.total < bj;
  const int at = (threadIdx.x & 63) & ~(Token::kLanes - 1);
  constexpr uint32_t kAll = Token::kLanes == 32 ? 0xffffffffu : 0xffffu;
  const uint32_t mine = (uint32_t)(__ballot(ok) >> at) & kAll;
  const int skip = mine ? 32 - __builtin_clz(mine) : 0;
  const uint32_t keep = (uint32_t)(__ballot(live && j < k && tok.rank >= skip) >> at) & kAll;
  if (live && j == 0) {
    n_skip[t] = skip;
    keep_mask[t] = keep;
  }
}

// ratios[i-1][t] = r_i of token t; grid: ceil(T / tokens per workgroup)
template <int KMAX>
__global__ __launch_bounds__(kMoeThreads) void moe_ratios_kernel(const float* __restrict__ w, int T, int k,
                                                                 float* ratios) {
  typedef MoeToken<KMAX> Token;
  const int j = threadIdx.x & (Token::kLanes - 1), tl = threadIdx.x / Token::kLanes;
  const int t = blockIdx.x * Token::kPerWorkgroup + tl;
  const float wj = w[(int64_t)min(t, T - 1) * k + min(j, k - 1)];
  const Token tok(wj, j, k);
  if (t < T && j < k - 1) ratios[(int64_t)j * T + t] = tok.prefix / tok.total;
}

// The value of 0-based rank `rank` (ascending) among vals[0 .. T): radix select on the bit patterns
// (the values are positive).  Every thread returns the value.
__device__ float select_rank(const float* __restrict__ vals, int T, uint32_t rank, uint32_t* hist, uint32_t* sh) {
  const int tid = threadIdx.x;
  uint32_t prefix = 0, need = rank;                       // `need` smaller keys with this prefix come first
  for (int shift = 24; shift >= 0; shift -= 8) {
    hist[tid] = 0;
    __syncthreads();
    const uint32_t hi_mask = shift == 24 ? 0u : (0xffffffffu << (shift + 8));
    for (int i = tid; i < T; i += 256) {
      const uint32_t key = __float_as_uint(vals[i]);
      if ((key & hi_mask) == prefix) atomicAdd(&hist[(key >> shift) & 0xff], 1u);
    }
    __syncthreads();
    if (tid == 0) {
      uint32_t below = 0;
      int bin = 0;
      for (; bin < 256; ++bin) {
        if (below + hist[bin] > need) break;
        below += hist[bin];
      }
      sh[0] = prefix | ((uint32_t)bin << shift);
      sh[1] = need - below;
    }
    __syncthreads();
    prefix = sh[0];
    need = sh[1];
    __syncthreads();
  }
  return __uint_as_float(prefix);
}

// grid: (k - 1); block: 256
__global__ __launch_bounds__(256) void moe_median_kernel(const float* __restrict__ ratios, int T, float* beta) {
  __shared__ uint32_t hist[256];
  __shared__ uint32_t sh[2];
  const float* col = ratios + (int64_t)blockIdx.x * T;
  const float hi = select_rank(col, T, (uint32_t)(T / 2), hist, sh);
  float med = hi;
  if ((T & 1) == 0) med = 0.5f * (select_rank(col, T, (uint32_t)(T / 2 - 1), hist, sh) + hi);
  if (threadIdx.x == 0) beta[blockIdx.x] = med;
}

// ---- acceptance / resampling -------------------------------------------------------------------
constexpr int kAccThreads = 1024;
constexpr int kAccWaves = kAccThreads / 64;
constexpr int kChunk = 256;                               // tokens per chunk: four per lane
constexpr int kMaxChunks = 2048;                          // sixteen segments of the scan

// Inclusive prefix sum over the 64 lanes with cross-lane operand moves only (no trip through LDS
// per step): shifts by 1, 2, 4, 8 inside each row of 16 lanes (lanes without a source add zero),
// then the last lane of row 0 / row 2 into rows 1 / 3, then the last lane of row 1 into rows 2, 3.
template <int CTRL, int ROW_MASK, bool BOUND>
__device__ __forceinline__ float lane_move(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, ROW_MASK, 0xf, BOUND));
}
__device__ __forceinline__ float wave_inclusive_sum_f(float v, int /*lane*/) {
  v += lane_move<0x111, 0xf, true>(v);    // row_shr:1
  v += lane_move<0x112, 0xf, true>(v);    // row_shr:2
  v += lane_move<0x114, 0xf, true>(v);    // row_shr:4
  v += lane_move<0x118, 0xf, true>(v);    // row_shr:8
  v += lane_move<0x142, 0xa, false>(v);   // row_bcast:15 -> rows 1, 3
  v += lane_move<0x143, 0xc, false>(v);   // row_bcast:31 -> rows 2, 3
  return v;
}

// Four consecutive floats on a four-byte boundary (a row of V floats starts on no better one when V is
// no multiple of four): one 16-byte load, which needs no more than that.
typedef float float4_u __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ float4 load4(const float* p) {
  const float4_u x = *reinterpret_cast<const float4_u*>(p);
  return make_float4(x.x, x.y, x.z, x.w);
}
__device__ __forceinline__ float4 residual4_of(float4 a, float4 d, bool from_target) {
  if (from_target) return a;
  return make_float4(fmaxf(0.f, a.x - d.x), fmaxf(0.f, a.y - d.y), fmaxf(0.f, a.z - d.z), fmaxf(0.f, a.w - d.w));
}

// Residual mass (Eq. 3) of tokens v .. v + 3 of the rejected position; tokens past V count nothing.
__device__ __forceinline__ float4 residual4(const float* __restrict__ pt, const float* __restrict__ pd, int v, int V,
                                            bool from_target) {
  float4 a = make_float4(0.f, 0.f, 0.f, 0.f), d = a;
  if (v + 3 < V) {
    a = load4(pt + v);
    d = load4(pd + v);
  } else {
    if (v < V) { a.x = pt[v]; d.x = pd[v]; }
    if (v + 1 < V) { a.y = pt[v + 1]; d.y = pd[v + 1]; }
    if (v + 2 < V) { a.z = pt[v + 2]; d.z = pd[v + 2]; }
    if (v + 3 < V) { a.w = pt[v + 3]; d.w = pd[v + 3]; }
  }
  return residual4_of(a, d, from_target);
}

// Four chunks of both distributions on their way: this lane's four tokens of each.
struct ChunkLoads { float4 a[4], d[4]; };

// Sums of chunks c_begin .. c_end - 1 by one wavefront: four whole chunks at a time, then what is left.
template <bool FROM_TARGET>
__device__ __forceinline__ void sum_chunks(const float* pt, const float* pd, int V, int c_begin, int c_end, int lane,
                                           float* csum) {
  auto sum_chunk = [&](int c, const float4& r) {
    const float incl = wave_inclusive_sum_f(((r.x + r.y) + r.z) + r.w, lane);
    if (lane == 63) csum[c] = incl;
  };
  const int whole = max(min(c_end, V / kChunk) - c_begin, 0) / 4;
  const float* pt_lane = pt + (int64_t)c_begin * kChunk + 4 * lane;
  const float* pd_lane = pd + (int64_t)c_begin * kChunk + 4 * lane;
  auto request = [&](int g, ChunkLoads& q) {
    const int at = g * (4 * kChunk);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      q.a[u] = load4(pt_lane + at + u * kChunk);
      q.d[u] = load4(pd_lane + at + u * kChunk);
    }
  };
  auto sum_up = [&](int g, const ChunkLoads& q) {
#pragma unroll
    for (int u = 0; u < 4; ++u) sum_chunk(c_begin + 4 * g + u, residual4_of(q.a[u], q.d[u], FROM_TARGET));
  };
  // (no branch between a request and its use inside the loop, which would make every wait a wait for
  // everything in flight, and no request behind the last group: the barrier that follows would wait for it, 1 us
  // of 9.6 for the 64 sequences of 32 000 tokens, whose wavefronts have two groups)
  ChunkLoads q0, q1;
  if (whole >= 2) {
    request(0, q0);
    request(1, q1);
    int g = 0;
    for (; g + 3 < whole; g += 2) {
      sum_up(g, q0);
      request(g + 2, q0);
      sum_up(g + 1, q1);
      request(g + 3, q1);
    }
    sum_up(g, q0);
    const bool third = g + 3 == whole;
    if (third) request(g + 2, q0);
    sum_up(g + 1, q1);
    if (third) sum_up(g + 2, q0);
  } else if (whole == 1) {
    request(0, q0);
    sum_up(0, q0);
  }
  for (int c = c_begin + 4 * whole; c < c_end; ++c) sum_chunk(c, residual4(pt, pd, c * kChunk + 4 * lane, V, FROM_TARGET));
}

// The scan of the chunk sums by one wavefront.  128 sums make a segment, two per lane; a lane's pair,
// the lanes of a segment and the segments are added in this order, so that the intervals
// [lower, upper) of pairs are built from the same sums wherever they are formed: one's upper bound is
// the next one's lower bound bit for bit, and exactly one pair holds the target.
struct ChunkScan {
  float total;
  float before;                        // lane s: sum of the segments in front of segment s
  __device__ __forceinline__ void sum_up(const float* csum, int n_chunks, int lane) {
    const int segments = (n_chunks + 127) / 128;
    float run = 0.f;
    before = 0.f;
#pragma unroll 4
    for (int s = 0; s < segments; ++s) {
      const float2 c = *reinterpret_cast<const float2*>(csum + 128 * s + 2 * lane);
      const float incl = wave_inclusive_sum_f(c.x + c.y, lane);
      if (lane == s) before = run;
      run += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(incl), 63));
    }
    total = run;
  }
  // The chunk that holds the target and the sum in front of it; the last chunk and zero where rounding (a
  // target that is not below the total) leaves it outside every interval.
  __device__ __forceinline__ int find(const float* csum, int n_chunks, float target, int lane, float& base) const {
    const int segments = (n_chunks + 127) / 128;
    base = 0.f;
    const uint64_t from = __ballot(lane < segments && before <= target);
    if (!from) return n_chunks - 1;
    const int s = 63 - __builtin_clzll(from);              // (the sums do not decrease)
    const float in_front = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(before), s));
    const float2 c = *reinterpret_cast<const float2*>(csum + 128 * s + 2 * lane);
    const float incl = wave_inclusive_sum_f(c.x + c.y, lane);
    const float prev = __shfl_up(incl, 1, 64);
    const float upper = in_front + incl, lower = lane == 0 ? in_front : in_front + prev;
    const uint64_t hit = __ballot(lower <= target && target < upper);
    if (!hit) return n_chunks - 1;
    const bool second = !(target < lower + c.x);
    const int l = __builtin_ctzll(hit);
    base = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(second ? lower + c.x : lower), l));
    return min(__builtin_amdgcn_readlane(2 * (64 * s + lane) + (second ? 1 : 0), l), n_chunks - 1);
  }
};

// grid: (B); block: 1024.  The vocabulary is cut into chunks of 256 consecutive tokens (a lane holds
// four, so a wavefront reads a chunk as one contiguous kilobyte per distribution); wavefront w sums
// the chunks of its contiguous share; one wavefront scans the chunk sums and walks the chunk the
// target mass falls in.  The intervals [lower, upper) are built so that
// one's upper bound is the next one's lower bound bit for bit: exactly one chunk and one lane match.
// Bound: 3.4 us that do not depend on the vocabulary (launch, the gamma tests, the scan, the walk), then
// what one compute unit takes in: one sequence 5.2 us at 32 000 tokens and 12.9 at 129 280, 45 bytes a clock.
// 64 sequences, all rejected: 7.0 and 21.9 us, 3.6 TB/s together.  The next four chunks are always on their way
// while four are summed.  With the scan by the whole workgroup and the choice of chunk and token handed on through
// LDS and barriers: 4.2 (1 000 tokens), 6.2 and 13.5 us for one sequence, 8.0 and 22.0 for the 64.
__global__ __launch_bounds__(kAccThreads) void accept_kernel(const float* __restrict__ p_target,
                                                             const float* __restrict__ p_draft,
                                                             const int32_t* __restrict__ draft_tokens,
                                                             const float* __restrict__ u_accept,
                                                             const float* __restrict__ u_resample, int gamma, int V,
                                                             int32_t* n_accepted, int32_t* resampled) {
  __shared__ __attribute__((aligned(8))) float csum[kMaxChunks];
  __shared__ int sh_n, sh_again;
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t seq = (int64_t)b * gamma;
  if (wave == 0) {
    bool rejected = false;
    if (lane < gamma) {
      const float u = u_accept[seq + lane];
      const int x = min(max(draft_tokens[seq + lane], 0), V - 1);
      const float pt = p_target[(seq + lane) * V + x], pd = p_draft[(seq + lane) * V + x];
      const float alpha = pd > 0.f ? fminf(1.0f, pt / pd) : 1.0f;                 // Eq. 2
      rejected = !(u < alpha);
    }
    const uint64_t rj = __ballot(rejected);
    if (lane == 0) sh_n = rj ? __builtin_ctzll(rj) : gamma;
  }
  __syncthreads();
  const int n = sh_n;
  if (n == gamma) {
    if (tid == 0) { n_accepted[b] = n; resampled[b] = -1; }
    return;
  }
  const float* pt = p_target + (seq + n) * V;
  const float* pd = p_draft + (seq + n) * V;
  const int n_chunks = (V + kChunk - 1) / kChunk;
  const int cpw = (n_chunks + kAccWaves - 1) / kAccWaves;
  const int c_begin = wave * cpw, c_end = min(c_begin + cpw, n_chunks);
  const float u_r = u_resample[b];
  if (tid < (n_chunks + 127) / 128 * 128 - n_chunks) csum[n_chunks + tid] = 0.f;     // the rest of the scan's last segment
  sum_chunks<false>(pt, pd, V, c_begin, c_end, lane, csum);
  __syncthreads();
  // What is left is a chain of short steps, by one wavefront: handed from step to step through LDS and a
  // barrier they cost several times what they compute.
  ChunkScan scan;
  if (wave == 0) {
    scan.sum_up(csum, n_chunks, lane);
    if (lane == 0) sh_again = scan.total > 0.f ? 0 : 1;
  }
  __syncthreads();
  const bool from_target = sh_again != 0;                 // the distributions coincide: resample from p_theta
  if (from_target) {
    sum_chunks<true>(pt, pd, V, c_begin, c_end, lane, csum);
    __syncthreads();
    if (wave == 0) scan.sum_up(csum, n_chunks, lane);
  }
  if (wave != 0) return;
  const float target = u_r * scan.total;
  float base;
  const int chunk = scan.find(csum, n_chunks, target, lane, base);
  const int v = chunk * kChunk + 4 * lane;
  const float4 r = residual4(pt, pd, v, V, from_target);
  const float incl = wave_inclusive_sum_f(((r.x + r.y) + r.z) + r.w, lane);
  const float prev = __shfl_up(incl, 1, 64);
  const float upper = base + incl;
  float c = lane == 0 ? base : base + prev;
  const uint64_t hit = __ballot(c <= target && target < upper);
  int mine = v + 3;
  c += r.x;
  if (c > target) mine = v;
  else if ((c += r.y) > target) mine = v + 1;
  else if ((c += r.z) > target) mine = v + 2;
  // (if rounding leaves the target just outside every lane's interval: the chunk's last token)
  int pick = min((chunk + 1) * kChunk, V) - 1;
  if (hit) pick = min(__builtin_amdgcn_readlane(mine, __builtin_ctzll(hit)), V - 1);
  if (lane == 0) { n_accepted[b] = n; resampled[b] = pick; }
}

// A kernel for k experts: the least KMAX that holds them (65 536 tokens of 17 experts: 16.5 us with KMAX = 32).
template <typename Launch>
void with_kmax(int k, Launch&& launch) {
  if (k <= 8) launch(std::integral_constant<int, 8>());
  else if (k <= 16) launch(std::integral_constant<int, 16>());
  else if (k <= 20) launch(std::integral_constant<int, 20>());
  else if (k <= 24) launch(std::integral_constant<int, 24>());
  else launch(std::integral_constant<int, 32>());
}
template <int KMAX>
dim3 moe_grid(int T) { return dim3((unsigned)((T + MoeToken<KMAX>::kPerWorkgroup - 1) / MoeToken<KMAX>::kPerWorkgroup)); }

size_t align256(size_t x) { return (x + 255) / 256 * 256; }

}  // namespace

extern "C" {

int svf_moe_skip(const float* w, int32_t T, int32_t k, int32_t m, const float* beta, int32_t* n_skip,
                 uint32_t* keep_mask, void* stream) {
  if (!w || !beta || !n_skip || !keep_mask) return SVF_ERR_NULL;
  if (T < 1 || k < 2 || k > 32) return SVF_ERR_SHAPE;
  if (m < 1 || m >= k) return SVF_ERR_BUDGET;
  hipStream_t st = static_cast<hipStream_t>(stream);
  with_kmax(k, [&](auto kmax) {
    hipLaunchKernelGGL(moe_skip_kernel<kmax>, moe_grid<kmax>(T), dim3(kMoeThreads), 0, st, w, T, k, m, beta, n_skip, keep_mask);
  });
  return hipGetLastError() == hipSuccess ? SVF_OK : SVF_ERR_HIP;
}

size_t svf_moe_calibrate_workspace_bytes(int32_t T, int32_t k) {
  if (T < 1 || k < 2 || k > 32) return 0;
  return align256((size_t)(k - 1) * T * sizeof(float));
}

int svf_moe_calibrate(const float* w_cal, int32_t T, int32_t k, float* beta, void* ws, size_t ws_bytes,
                      void* stream) {
  if (!w_cal || !beta) return SVF_ERR_NULL;
  if (T < 1 || k < 2 || k > 32) return SVF_ERR_SHAPE;
  if (!ws || reinterpret_cast<uintptr_t>(ws) % 256 || ws_bytes < svf_moe_calibrate_workspace_bytes(T, k))
    return SVF_ERR_WORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  float* ratios = static_cast<float*>(ws);
  with_kmax(k, [&](auto kmax) {
    hipLaunchKernelGGL(moe_ratios_kernel<kmax>, moe_grid<kmax>(T), dim3(kMoeThreads), 0, st, w_cal, T, k, ratios);
  });
  if (hipGetLastError() != hipSuccess) return SVF_ERR_HIP;
  hipLaunchKernelGGL(moe_median_kernel, dim3(k - 1), dim3(256), 0, st, ratios, T, beta);
  return hipGetLastError() == hipSuccess ? SVF_OK : SVF_ERR_HIP;
}

int svf_accept_resample(const float* p_target, const float* p_draft, const int32_t* draft_tokens,
                        const float* u_accept, const float* u_resample, int32_t B, int32_t gamma, int32_t V,
                        int32_t* n_accepted, int32_t* resampled, void* stream) {
  if (!p_target || !p_draft || !draft_tokens || !u_accept || !u_resample || !n_accepted || !resampled)
    return SVF_ERR_NULL;
  if (B < 1 || gamma < 1 || gamma > 64 || V < 1 || V > kMaxChunks * kChunk) return SVF_ERR_SHAPE;
  hipLaunchKernelGGL(accept_kernel, dim3(B), dim3(kAccThreads), 0, static_cast<hipStream_t>(stream), p_target, p_draft,
                     draft_tokens, u_accept, u_resample, gamma, V, n_accepted, resampled);
  return hipGetLastError() == hipSuccess ? SVF_OK : SVF_ERR_HIP;
}

}  // extern "C"
