// Retrieval: block scores and the kept blocks, in one launch or two (Sec. 3.1, Eq. 5 and the selection rule), with
// one rule of Sec. 3.1 exchanged where the caller asks for it.
//
//   scores  the first draft token's score of every block: with the query averaged over the query heads of
//           a KV head (the main path's rule), or PER QUERY HEAD, against the mean key (Eq. 5) or against
//           the per-channel minimum / maximum of the block's keys (Quest's summary, which Sec. 3.1 starts
//           from:  sum_c max(q_c min_c, q_c max_c) >= q . k for every key of the block), the query heads
//           of a KV head combined by their mean or their maximum.  Summaries are fp32 or bf16.  Eight lanes
//           own a block, 16 channels each (d = 128), fixed order of the arithmetic; the summaries are read
//           once whatever the number of query heads.
//   select  top-N over the blocks of a KV head, or over all (KV head, block) pairs of a sequence (Eq. 6
//           counts its budget over the H KV heads), by the workgroup that is the last of its KV head
//           (or sequence) to have stored its scores, or in a launch of its own (selection_of): radix select over
//           keys in registers, then one ordered compaction.
//
// What bounds it: latency.  The summaries are a few MB; the rest is a chain of launch, query, scores, exchange,
// three or four radix digits of one barrier each, compaction.  128 blocks per workgroup, so that many compute
// units score; us per call, against scores and selection as two launches of their own: 32 heads of 512 blocks (min/max
// bf16, group maximum) 13.3 -> 8.7, mean bf16 10.5 -> 6.9, 16 heads of 1024 16.0 -> 9.3, of 2048 22.4 -> 11.4, 8 heads of 250
// 11.1 -> 7.0; one selection over all heads, four sequences of 8 x 512 15.0 -> 12.3, one of 8 x 1024 18.7 -> 15.0.
#include <hip/hip_bf16.h>

#include "svf_device.h"

namespace svf {

namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr int kScoreThreads = 256;     // of a launch that only scores
constexpr int kScorePasses = 4;        // its blocks per lane group
constexpr int kBlocksPerGroup = kThreads / kScoreLanes;   // blocks per workgroup that scores
static_assert(kScorePasses * kScoreThreads == kThreads, "the same blocks per workgroup");
constexpr int kHeadsPerRound = 8;      // query heads staged in LDS at a time
constexpr int kKeys = 8;               // keys per thread of a selection in the launch that scores
constexpr int kManyKeys = 32;          // the most in a launch of its own
constexpr int kMaxHeads = 256;         // KV heads of one selection

__device__ __forceinline__ float4 load4(const float* p) { return *reinterpret_cast<const float4*>(p); }
__device__ __forceinline__ float4 load4(const __hip_bfloat16* p) {
  const uint2 w = *reinterpret_cast<const uint2*>(p);
  return make_float4(__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u), __uint_as_float(w.y << 16),
                     __uint_as_float(w.y & 0xffff0000u));
}

// sum over this lane's channels of max(q * min, q * max), then over the lane group
template <int NCH>
__device__ __forceinline__ float bound_score(const float4 (&mn)[NCH], const float4 (&mx)[NCH], const float4 (&q)[NCH]) {
  float acc = 0.f;
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    acc += fmaxf(q[i].x * mn[i].x, q[i].x * mx[i].x);
    acc += fmaxf(q[i].y * mn[i].y, q[i].y * mx[i].y);
    acc += fmaxf(q[i].z * mn[i].z, q[i].z * mx[i].z);
    acc += fmaxf(q[i].w * mn[i].w, q[i].w * mx[i].w);
  }
  return lane8_sum(acc);
}

// How a block is scored (VariantParams::mean_query, minmax, group_max).
enum Rule { kMeanQuery, kMeanOfHeads, kMaxOfHeads, kBoundMeanOfHeads, kBoundMaxOfHeads };

// What a selection over KEYS keys per thread needs in LDS.
// COPIES of a digit's histogram: lanes l, l + COPIES, ... count in one of them (a bin of all of them in different banks).
template <int COPIES>
struct Counts {
  static constexpr int kCopies = COPIES, kStride = COPIES == 1 ? 256 : 260;
  uint32_t hist[4][COPIES * kStride];
  uint32_t low[kWaves], high[kWaves], top[kWaves];   // of a wavefront's keys: smallest, largest below the top key, top keys
};
// (With many keys per thread, the adds to the few bins that most scores share are what a digit takes: 32 768 pairs
// 55.4 us a retrieval with one copy, 51.7 with two, 49.8 with four, 49.6 with eight.)
template <int KEYS, int COPIES>
struct Scratch : Counts<COPIES> {
  uint32_t seg[KEYS * kWaves];           // larger keys (low half) and equal keys of 64 consecutive keys
  uint32_t head_rank[kMaxHeads + 1];     // kept pairs in front of a head's first
  int32_t sel[kMaxGatherBlocks];         // kept block ids, for the gather list
};

constexpr uint32_t kTopKey = 0xffffffffu;  // of a block that is always kept
constexpr uint32_t kAllEqual = 0xffffffffu;

// Minimum / maximum over the 64 lanes, by cross-lane operand modifiers only (see wave_inclusive_sum; lanes
// without a source keep their own value).
template <bool MAX>
__device__ __forceinline__ uint32_t wave_extreme(uint32_t x) {
#define SVF_STEP(CTRL, ROWS)                                                                            \
  {                                                                                                     \
    const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, CTRL, ROWS, 0xf, false);   \
    x = MAX ? max(x, o) : min(x, o);                                                                    \
  }
  SVF_STEP(0x111, 0xf)   // row_shr:1
  SVF_STEP(0x112, 0xf)   // row_shr:2
  SVF_STEP(0x114, 0xf)   // row_shr:4
  SVF_STEP(0x118, 0xf)   // row_shr:8
  SVF_STEP(0x142, 0xa)   // row_bcast:15 -> rows 1, 3
  SVF_STEP(0x143, 0xc)   // row_bcast:31 -> rows 2, 3
#undef SVF_STEP
  return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}

// One digit of the radix select: finds the bin of hist that the need-th largest key lies in.  Every wavefront scans
// the 256 bins for itself, lane l bins 255 - 4l (in .w) down to 252 - 4l (in .x).  need becomes what is still wanted
// from inside the bin; true if that is all of it.
template <int COPIES, int STRIDE>
__device__ __forceinline__ bool pick_bin(const uint32_t (&hist)[COPIES * STRIDE], int lane, uint32_t& need, uint32_t& bin_out) {
  uint4 hq = *reinterpret_cast<const uint4*>(&hist[252 - 4 * lane]);
#pragma unroll
  for (int c = 1; c < COPIES; ++c) {
    const uint4 other = *reinterpret_cast<const uint4*>(&hist[c * STRIDE + 252 - 4 * lane]);
    hq.x += other.x; hq.y += other.y; hq.z += other.z; hq.w += other.w;
  }
  const uint32_t own = hq.x + hq.y + hq.z + hq.w;
  const uint32_t incl = wave_inclusive_sum(own);
  uint32_t run = incl - own;
  const uint64_t cross = __ballot(incl >= need && run < need);         // one lane
  uint32_t bin = 255u - 4u * (uint32_t)lane, in_bin = hq.w;
  if (run + hq.w < need) {
    run += hq.w; --bin; in_bin = hq.z;
    if (run + hq.z < need) {
      run += hq.z; --bin; in_bin = hq.y;
      if (run + hq.y < need) { run += hq.y; --bin; in_bin = hq.x; }
    }
  }
  const int src = __builtin_ctzll(cross);
  bin_out = (uint32_t)__builtin_amdgcn_readlane((int)bin, src);
  need -= (uint32_t)__builtin_amdgcn_readlane((int)run, src);
  return need == (uint32_t)__builtin_amdgcn_readlane((int)in_bin, src);
}

// The key of the weakest of the keep_n >= 1 largest of N keys; need: how many keys equal to it are kept (kAllEqual:
// all, and the key may then be smaller than the smallest kept one).  A histogram per digit in LDS (all zeroed by
// the caller, a barrier since), one barrier per digit.
// One key per thread (N <= 1024): the digits are the key's bytes.  Scores share their sign and most of their
// exponent, so the first byte tells few of them apart, and a wavefront's adds to one bin go one lane at a
// time: the lanes that share the first lane's bin are counted with one add.
template <typename Counts>
__device__ __forceinline__ uint32_t threshold_of(uint32_t key, Counts* sc, int N, uint32_t keep_n, int tid, int lane, uint32_t& need) {
  uint32_t prefix = 0;
  need = keep_n;
#pragma unroll
  for (int pass = 0; pass < 4; ++pass) {
    const int shift = 24 - 8 * pass;
    const bool in = tid < N && (pass == 0 || (key ^ prefix) >> ((shift + 8) & 31) == 0);
    const uint32_t bin = (key >> shift) & 0xffu;
    const uint64_t m = __ballot(in);
    if (m != 0) {                                        // (uniform)
      const int first = __builtin_ctzll(m);
      const uint32_t bin0 = (uint32_t)__builtin_amdgcn_readlane((int)bin, first);
      const uint64_t same = __ballot(in && bin == bin0);
      if (lane == first) atomicAdd(&sc->hist[pass][bin0], (uint32_t)__popcll(same));
      else if (in && bin != bin0) atomicAdd(&sc->hist[pass][bin], 1u);
    }
    __syncthreads();
    uint32_t picked;
    const bool whole = pick_bin<Counts::kCopies, Counts::kStride>(sc->hist[pass], lane, need, picked);
    prefix |= picked << shift;
    if (whole) {
      need = kAllEqual;
      break;
    }
  }
  return prefix;
}
// Several keys per thread (thread t: keys t, t + 1024, ...): the digits are taken from the top of the keys' range,
// which saves one or two of them and spreads the adds, and costs a pass and a barrier: four sequences of 4096
// keys 13.4 -> 12.3 us a call, one of 8192 keys 17.2 -> 15.2 (32 heads of 512 keys 9.0 -> 9.1).
template <int KEYS, typename Counts>
__device__ __forceinline__ uint32_t threshold_of(const uint32_t (&key)[KEYS], Counts* sc, int N, uint32_t keep_n, int tid, int lane,
                                                 int wave, uint32_t& need) {
  uint32_t low = kTopKey, high = 0u, top = 0u;           // (top keys stand apart, or the range would be all there is)
#pragma unroll
  for (int u = 0; u < KEYS; ++u) {
    if (u * kThreads >= N) break;                        // (uniform)
    const bool in = u * kThreads + tid < N, is_top = in && key[u] == kTopKey;
    top += (uint32_t)__popcll(__ballot(is_top));
    low = min(low, in ? key[u] : kTopKey);
    high = max(high, in && !is_top ? key[u] : 0u);
  }
  low = wave_extreme<false>(low);
  high = wave_extreme<true>(high);
  if (lane == 0) {
    sc->low[wave] = low;
    sc->high[wave] = high;
    sc->top[wave] = top;
  }
  __syncthreads();
  {
    const int w = lane & (kWaves - 1);
    static_assert((kWaves & (kWaves - 1)) == 0 && kWaves <= 64, "a lane per wavefront");
    low = wave_extreme<false>(sc->low[w]);
    high = wave_extreme<true>(sc->high[w]);
    top = (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_sum(lane < kWaves ? sc->top[w] : 0u), 63);
  }
  need = keep_n;
  if (top >= keep_n) return kTopKey;
  need -= top;
  uint32_t prefix = 0;                                   // of key - low, the bits from `shift` up
  int shift = 32 - __builtin_clz((high - low) | 1u);
#pragma unroll 1
  for (int pass = 0; pass < 4; ++pass) {
    const int width = min(shift, 8);
    shift -= width;
#pragma unroll
    for (int u = 0; u < KEYS; ++u) {
      if (u * kThreads >= N) break;
      const uint32_t rel = key[u] - low;
      if (u * kThreads + tid < N && key[u] != kTopKey && (uint64_t)(rel ^ prefix) >> (shift + width) == 0)
        atomicAdd(&sc->hist[pass][lane % Counts::kCopies * Counts::kStride + ((rel >> shift) & ((1u << width) - 1u))], 1u);
    }
    __syncthreads();
    uint32_t picked;
    const bool whole = pick_bin<Counts::kCopies, Counts::kStride>(sc->hist[pass], lane, need, picked);
    prefix |= picked << shift;
    if (whole) {
      need = kAllEqual;
      break;
    }
    if (shift == 0) break;
  }
  return low + prefix;
}

// PART: what a launch does.  Scores and selection, by the workgroup that arrives last; or the one or the other.
enum Part { kBoth, kScoresOnly, kSelectionOnly };

// The scores alone take four blocks per lane group of a quarter of the threads: as many bytes on their way with fewer
// wavefronts, which pays where the workgroups come in rounds.  A selection alone, us per retrieval with the scores'
// launch, against one that reads the scores again in every pass: one budget over 8 x 1025 pairs 36.7 -> 19.9,
// 8 x 2048 41.4 -> 28.3, 8 x 4096 72.8 -> 46.9, 128 x 200 284 -> 45; per head, 8 heads of 9000 blocks 65 -> 23, of
// 32 768 231 -> 61.
// grid: (ceil(nb_max / 128), Hkv, B); the selection alone: (1, 1 for all heads or Hkv, B)
template <typename QT, typename RT, int D, int RULE, int PART, int KEYS>
__global__ __launch_bounds__(PART == kScoresOnly ? kScoreThreads : kThreads) void retrieve_kernel(VariantParams p) {
  constexpr int kOwnThreads = PART == kScoresOnly ? kScoreThreads : kThreads;
  constexpr int kPasses = PART == kScoresOnly ? kScorePasses : 1;      // blocks per lane group
  constexpr int kBlocksPerPass = kOwnThreads / kScoreLanes;
  constexpr int LPB = kScoreLanes;
  constexpr int NCH = D / (4 * LPB);
  constexpr bool MINMAX = RULE == kBoundMeanOfHeads || RULE == kBoundMaxOfHeads;
  constexpr bool GMAX = RULE == kMaxOfHeads || RULE == kBoundMaxOfHeads;
  constexpr int ROWS = MINMAX ? 2 : 1;
  __shared__ __attribute__((aligned(16))) float qs[RULE == kMeanQuery ? 1 : kHeadsPerRound][D];
  __shared__ uint32_t s_keys[kBlocksPerGroup];            // (one workgroup alone) the keys as they are formed
  __shared__ __attribute__((aligned(16))) Scratch<KEYS, PART == kBoth ? 1 : 4> s_scratch;
  __shared__ int s_last;

  const int b = blockIdx.z;
  const int tid = threadIdx.x, sub = tid % LPB;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = p.Hq / p.Hkv;
  auto* const sc = &s_scratch;
  const bool alone = gridDim.x == 1 && (!p.all_heads || p.Hkv == 1);   // one workgroup scores all it selects from
  int L, nb;
  if constexpr (PART != kSelectionOnly) {
    // All loads go out before anything waits.  Summaries unconditionally (rows past the sequence's last block
    // exist in the buffer; their result is discarded).
    const int h = blockIdx.y;
    float4 r[kPasses][ROWS][NCH];
    int jj[kPasses];
    const QT* const q0 = static_cast<const QT*>(p.q) + ((int64_t)b * p.gamma * p.Hq + (int64_t)h * G) * D;
    QueryHeads<QT> qh;
    if constexpr (RULE == kMeanQuery) qh = load_query_heads<QT>(q0 + tid % D, G, D);
#pragma unroll
    for (int u = 0; u < kPasses; ++u) {
      const int j = (blockIdx.x * kPasses + u) * kBlocksPerPass + tid / LPB;
      jj[u] = j;
      const RT* row = static_cast<const RT*>(p.summaries) + ((((int64_t)b * p.Hkv + h) * p.nb_max + min(j, p.nb_max - 1)) * ROWS) * D + sub * 4;
#pragma unroll
      for (int w = 0; w < ROWS; ++w)
#pragma unroll
        for (int i = 0; i < NCH; ++i) r[u][w][i] = load4(row + w * D + i * 4 * LPB);
    }
    L = clamped_len(p.seq_lens, b, p.max_seq_len);
    nb = (L + p.block_size - 1) / p.block_size;
    if constexpr (PART == kBoth)
      for (int i = tid; i < 4 * 256; i += kThreads) (&sc->hist[0][0])[i] = 0;

    float acc[kPasses];
#pragma unroll
    for (int u = 0; u < kPasses; ++u) acc[u] = GMAX ? -__builtin_inff() : 0.f;
    if constexpr (RULE == kMeanQuery) {
      if (tid < D) qs[0][tid] = mean_query_channel<QT>(qh, q0 + tid % D, G, D);
      __syncthreads();
      float4 qv[NCH];
#pragma unroll
      for (int i = 0; i < NCH; ++i) qv[i] = *reinterpret_cast<const float4*>(&qs[0][sub * 4 + i * 4 * LPB]);
#pragma unroll
      for (int u = 0; u < kPasses; ++u) acc[u] = block_score<NCH>(r[u][0], qv);
    } else {
      for (int g0 = 0; g0 < G; g0 += kHeadsPerRound) {
        const int ng = min(kHeadsPerRound, G - g0);
        if (g0 > 0) __syncthreads();                      // the round before has been read
        for (int idx = tid; idx < ng * D; idx += kOwnThreads) (&qs[0][0])[idx] = query_value(q0[(int64_t)g0 * D + idx]);
        __syncthreads();
        for (int g = 0; g < ng; ++g) {
          float4 qv[NCH];
#pragma unroll
          for (int i = 0; i < NCH; ++i) qv[i] = *reinterpret_cast<const float4*>(&qs[g][sub * 4 + i * 4 * LPB]);
#pragma unroll
          for (int u = 0; u < kPasses; ++u) {
            float s;
            if constexpr (MINMAX) s = bound_score<NCH>(r[u][0], r[u][ROWS - 1], qv);
            else s = block_score<NCH>(r[u][0], qv);
            acc[u] = GMAX ? fmaxf(acc[u], s) : acc[u] + s;
          }
        }
      }
      if constexpr (!GMAX) {
#pragma unroll
        for (int u = 0; u < kPasses; ++u) acc[u] = acc[u] / (float)G;
      }
    }
#pragma unroll
    for (int u = 0; u < kPasses; ++u)
      if (sub == 0 && jj[u] < p.nb_max) {
        const float v = jj[u] < nb ? acc[u] + 0.0f : 0.0f;
        float* const to = p.scores + ((int64_t)b * p.Hkv + h) * p.nb_max + jj[u];
        if constexpr (PART == kScoresOnly) {
          *to = v;
          continue;
        }
        // (write-through: the workgroup that selects may run on another XCD)
        __hip_atomic_store(to, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (alone) s_keys[jj[u]] = (jj[u] < p.n_sink || jj[u] >= nb - p.n_local) ? kTopKey : score_key(v);
      }
  } else {
    L = clamped_len(p.seq_lens, b, p.max_seq_len);
    nb = (L + p.block_size - 1) / p.block_size;
    for (int i = tid; i < (int)(sizeof(sc->hist) / 4); i += kThreads) (&sc->hist[0][0])[i] = 0;
  }
  if constexpr (PART == kScoresOnly) return;

  // ---- the last workgroup of the KV head (or of the sequence) selects ----
  const int h0 = p.all_heads ? 0 : blockIdx.y, heads = p.all_heads ? p.Hkv : 1;
  const int N = heads * nb;
  // head of pair i: a multiplication by 2^32 / nb, rounded up (exact: i, nb <= 32768)
  const uint32_t per_nb = nb > 1 ? 0xffffffffu / (uint32_t)nb + 1u : 0u;
  auto head_of = [&](int i) { return heads == 1 ? 0 : (nb > 1 ? (int)__umulhi((uint32_t)i, per_nb) : i); };
  uint32_t key[KEYS];
  if constexpr (PART == kBoth) {
#pragma unroll
    for (int u = 0; u < KEYS; ++u) key[u] = 0u;
  }
  if (PART == kSelectionOnly || !alone) {
    if constexpr (PART == kBoth) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // this wavefront's scores have been acknowledged
      __syncthreads();
      if (tid == 0) {
        uint64_t* const arrivals = p.tickets + ((int64_t)b * p.Hkv + h0) * kTicketWords + 2;
        const uint64_t of = (uint64_t)gridDim.x * heads;
        const uint64_t prev = __hip_atomic_fetch_add(arrivals, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_last = prev == of - 1;
        if (s_last) __hip_atomic_store(arrivals, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      __syncthreads();
      if (!s_last) return;
    }
    // scores of pair i = h * nb + j, all in flight at once
    const float* const from = p.scores + ((int64_t)b * p.Hkv + h0) * p.nb_max;
    float v[KEYS];
    int j[KEYS];
#pragma unroll
    for (int u = 0; u < KEYS; ++u) {
      if (u * kThreads >= N) break;                      // (uniform)
      const int i = min(u * kThreads + tid, N - 1), h = head_of(i);
      j[u] = i - h * nb;
      v[u] = __hip_atomic_load(from + (int64_t)h * p.nb_max + j[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
#pragma unroll
    for (int u = 0; u < KEYS; ++u) {
      if (u * kThreads >= N) continue;
      key[u] = (j[u] < p.n_sink || j[u] >= nb - p.n_local) ? kTopKey : score_key(v[u]);
    }
  }
  const uint32_t keep_n = (uint32_t)min(N, p.all_heads ? p.n_total : p.k_blocks);
  if (tid <= heads) sc->head_rank[tid] = keep_n;          // heads behind the last pair (an empty sequence: all)
  __syncthreads();
  if (PART == kBoth && alone && tid < N) key[0] = s_keys[tid];
  uint32_t need = 0, tau = kTopKey;
  if (keep_n > 0)
    tau = N <= kThreads ? threshold_of(key[0], sc, N, keep_n, tid, lane, need) : threshold_of<KEYS>(key, sc, N, keep_n, tid, lane, wave, need);
  const bool all_equal = need == kAllEqual;              // (a selection that cuts through equal keys is rare)

  // Per 64 keys the number of larger and of equal ones, and one scan over them (neither sum exceeds 32768): a
  // key's rank among the kept ones is then known, and with it, at the pairs that begin a head, where that
  // head's list starts.
  auto look = [&](int u, uint64_t& gt, uint64_t& eq) {
    const bool in = u * kThreads + tid < N;
    gt = __ballot(in && (all_equal ? key[u] >= tau : key[u] > tau));
    eq = all_equal ? 0ull : __ballot(in && key[u] == tau);
  };
#pragma unroll
  for (int u = 0; u < KEYS; ++u) {
    if (u * kThreads >= N) break;
    uint64_t gt, eq;
    look(u, gt, eq);
    if (lane == 0) sc->seg[u * kWaves + wave] = (uint32_t)__popcll(gt) | ((uint32_t)__popcll(eq) << 16);
  }
  __syncthreads();
  // (every wavefront scans them for itself: lane l holds segments kPer l .. kPer l + kPer - 1, and of their sums
  // keeps the one in front of the segment that the wavefront's own are: u * kWaves + wave)
  constexpr int kPer = KEYS * kWaves / 64;
  static_assert(kWaves % kPer == 0, "a wavefront's segments have the same place in every lane");
  uint32_t in_front;
  {
    const int segments = (N + kThreads - 1) / kThreads * kWaves;
    uint32_t sum = 0, before = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      if (i == wave % kPer) before = sum;
      sum += kPer * lane + i < segments ? sc->seg[kPer * lane + i] : 0u;
    }
    in_front = wave_inclusive_sum(sum) - sum + before;
  }
  uint32_t rank[KEYS];
  uint32_t kept = 0;                                       // bit u
  static_assert(KEYS <= 32, "a bit per key");
#pragma unroll
  for (int u = 0; u < KEYS; ++u) {
    if (u * kThreads >= N) break;
    uint64_t gt, eq;
    look(u, gt, eq);
    const uint32_t s = (uint32_t)__builtin_amdgcn_readlane((int)in_front, (u * kWaves + wave) / kPer);
    rank[u] = __builtin_amdgcn_mbcnt_hi((uint32_t)(gt >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)gt, s & 0xffffu));
    bool keep = (gt >> lane) & 1ull;
    if (!all_equal) {
      const uint32_t eq_before = __builtin_amdgcn_mbcnt_hi((uint32_t)(eq >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)eq, s >> 16));
      rank[u] += min(eq_before, need);
      keep |= ((eq >> lane) & 1ull) && eq_before < need;
    }
    if (keep) kept |= 1u << u;
    const int i = u * kThreads + tid, h = head_of(i);
    if (heads > 1 && i < N && i == h * nb) sc->head_rank[h] = rank[u];
  }
  if (heads > 1) __syncthreads();
  int32_t* const out = p.sel_idx + ((int64_t)b * p.Hkv + h0) * p.k_blocks;
#pragma unroll
  for (int u = 0; u < KEYS; ++u) {
    if (u * kThreads >= N) break;
    if (!((kept >> u) & 1u)) continue;
    const int i = u * kThreads + tid, h = head_of(i);
    const uint32_t pos = heads == 1 ? rank[u] : rank[u] - sc->head_rank[h];
    if (pos < (uint32_t)p.k_blocks) out[(int64_t)h * p.k_blocks + pos] = i - h * nb;
    if (heads == 1 && pos < (uint32_t)kMaxGatherBlocks) sc->sel[pos] = i;
  }
  for (int h = wave; h < heads; h += kWaves) {
    const int cnt = heads == 1 ? (int)keep_n : min((int)(sc->head_rank[h + 1] - sc->head_rank[h]), p.k_blocks);
    for (int i = cnt + lane; i < p.k_blocks; i += 64) out[(int64_t)h * p.k_blocks + i] = -1;
    if (lane == 0) p.sel_cnt[(int64_t)b * p.Hkv + h0 + h] = cnt;
  }
  // Gather list: where the K row of every fourth selected-token slot sits in the pool, and how many of its
  // four slots hold a real token (block and page sizes are multiples of four, so the four slots share a block
  // and a page).
  if (p.gather) {                                        // (one KV head at a time)
    __syncthreads();
    uint64_t* const gl = p.gather + ((int64_t)b * p.Hkv + h0) * p.gather_groups;
    for (int e = tid; e < p.gather_groups; e += kThreads) {
      const int slot0 = 4 * e, bi = slot0 / p.block_size;
      uint64_t entry = 0;
      if (bi < (int)keep_n) {
        const int tok0 = sc->sel[bi] * p.block_size + (slot0 - bi * p.block_size);
        const int nv = min(max(L - tok0, 0), 4);
        if (nv > 0) {
          const int64_t off = (token_offset(p.kv, p.table, b, tok0) + (int64_t)h0 * p.kv.stride_head) * 2;
          entry = ((uint64_t)off & kGatherOffsetMask) | ((uint64_t)nv << kGatherCountShift);
        }
      }
      gl[e] = entry;
    }
  }
}

template <typename QT, typename RT, int D, int RULE>
void launch_kernel(const VariantParams& p, bool select, hipStream_t st) {
  const dim3 grid((p.nb_max + kBlocksPerGroup - 1) / kBlocksPerGroup, p.Hkv, p.B);
  if (select) hipLaunchKernelGGL((retrieve_kernel<QT, RT, D, RULE, kBoth, kKeys>), grid, dim3(kThreads), 0, st, p);
  else hipLaunchKernelGGL((retrieve_kernel<QT, RT, D, RULE, kScoresOnly, kKeys>), grid, dim3(kScoreThreads), 0, st, p);
}
template <typename QT, typename RT, int D>
void launch_rule(const VariantParams& p, bool select, hipStream_t st) {
  if (p.minmax) {
    if (p.group_max) launch_kernel<QT, RT, D, kBoundMaxOfHeads>(p, select, st);
    else launch_kernel<QT, RT, D, kBoundMeanOfHeads>(p, select, st);
  } else if (p.mean_query) {                               // (fp32 summaries)
    launch_kernel<QT, float, D, kMeanQuery>(p, select, st);
  } else {
    if (p.group_max) launch_kernel<QT, RT, D, kMaxOfHeads>(p, select, st);
    else launch_kernel<QT, RT, D, kMeanOfHeads>(p, select, st);
  }
}
template <typename QT, typename RT>
void launch_d(const VariantParams& p, bool select, hipStream_t st) {
  if (p.d == 64) launch_rule<QT, RT, 64>(p, select, st);
  else launch_rule<QT, RT, 128>(p, select, st);
}

// ---- more pairs than a workgroup's registers hold ------------------------------------------------
constexpr int kGThreads = 1024;
constexpr int kGWaves = kGThreads / 64;

// Top-N over the (KV head, block) pairs of a sequence: the scores are read again in every pass.
// grid: (B)
__global__ __launch_bounds__(kGThreads) void select_global_kernel(VariantParams p) {
  __shared__ uint32_t hist[256];
  __shared__ uint32_t sh_prefix, sh_need;
  __shared__ uint32_t wave_eq[kGWaves], wave_sel[kGWaves];
  __shared__ uint32_t base_eq, base_sel;

  const int b = blockIdx.x;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int L = clamped_len(p.seq_lens, b, p.max_seq_len);
  const int nb = (L + p.block_size - 1) / p.block_size;
  const int64_t total = (int64_t)p.Hkv * nb;
  const uint32_t keep_n = (uint32_t)(total < p.n_total ? total : p.n_total);
  const float* sc = p.scores + (int64_t)b * p.Hkv * p.nb_max;
  int32_t* out = p.sel_idx + (int64_t)b * p.Hkv * p.k_blocks;

  auto key_of = [&](int h, int j) -> uint32_t {
    if (j < p.n_sink || j >= nb - p.n_local) return 0xffffffffu;
    return score_key(sc[(int64_t)h * p.nb_max + j]);
  };

  // radix select: key of the keep_n-th largest pair
  if (tid == 0) { sh_prefix = 0; sh_need = keep_n; }
  for (int shift = 24; shift >= 0; shift -= 8) {
    if (tid < 256) hist[tid] = 0;
    __syncthreads();
    const uint32_t prefix = sh_prefix;
    const uint32_t need = sh_need;
    const uint32_t hi_mask = shift == 24 ? 0u : (0xffffffffu << (shift + 8));
    for (int h = 0; h < p.Hkv; ++h)
      for (int j = tid; j < nb; j += kGThreads) {
        const uint32_t k = key_of(h, j);
        if ((k & hi_mask) == prefix) atomicAdd(&hist[(k >> shift) & 0xff], 1u);
      }
    __syncthreads();
    // thread t < 256 looks at bin 255 - t: the inclusive prefix sum over those threads counts the
    // keys in this bin and all higher ones; exactly one thread sees the count cross `need`
    uint32_t hcount = 0, incl = 0;
    if (tid < 256) {                                     // whole wavefronts
      hcount = hist[255 - tid];
      incl = wave_inclusive_sum(hcount);
      if (lane == 63) wave_eq[wave] = incl;
    }
    __syncthreads();
    if (tid < 256) {
      for (int w = 0; w < wave; ++w) incl += wave_eq[w];
      const uint32_t above = incl - hcount;
      if (incl >= need && above < need) {
        sh_need = need - above;                          // (every thread read sh_need before the last barrier)
        sh_prefix = prefix | ((uint32_t)(255 - tid) << shift);
      }
    }
    __syncthreads();
  }
  const uint32_t tau = sh_prefix;            // key of the weakest kept pair
  const uint32_t need_eq = sh_need;          // pairs equal to tau that are kept (lowest head, then block, first)

  // ordered sweep, head by head: a head's kept blocks come out ascending, pairs equal to tau are
  // kept in (head, block) order until need_eq of them are
  if (tid == 0) base_eq = 0;
  for (int h = 0; h < p.Hkv; ++h) {
    if (tid == 0) base_sel = 0;
    __syncthreads();
    for (int j0 = 0; j0 < nb; j0 += kGThreads) {
      const int j = j0 + tid;
      const uint32_t k = j < nb ? key_of(h, j) : 0u;
      const bool is_eq = keep_n > 0 && j < nb && k == tau;
      const bool is_gt = keep_n > 0 && j < nb && k > tau;
      const uint64_t m_eq = __ballot(is_eq);
      const uint64_t m_gt = __ballot(is_gt);
      if (lane == 0) { wave_eq[wave] = (uint32_t)__popcll(m_eq); wave_sel[wave] = (uint32_t)__popcll(m_gt); }
      __syncthreads();
      const uint64_t below = (1ull << lane) - 1ull;
      uint32_t eq_before = base_eq + (uint32_t)__popcll(m_eq & below), gt_before = (uint32_t)__popcll(m_gt & below);
      uint32_t eq_all = base_eq;
      for (int w = 0; w < kGWaves; ++w) {
        if (w < wave) { eq_before += wave_eq[w]; gt_before += wave_sel[w]; }
        eq_all += wave_eq[w];
      }
      // position = kept pairs in front: all larger ones, and the equal ones still inside need_eq
      const uint32_t eq_kept_before = min(eq_before, need_eq) - min(base_eq, need_eq);
      const bool keep = is_gt || (is_eq && eq_before < need_eq);
      const uint32_t pos = base_sel + gt_before + eq_kept_before;
      if (keep && pos < (uint32_t)p.k_blocks) out[(int64_t)h * p.k_blocks + pos] = j;
      __syncthreads();                                   // the per-wavefront counts have been read
      if (tid == 0) {
        uint32_t gt_all = 0;
        for (int w = 0; w < kGWaves; ++w) gt_all += wave_sel[w];
        base_sel += gt_all + (min(eq_all, need_eq) - min(base_eq, need_eq));
        base_eq = eq_all;
      }
      __syncthreads();
    }
    const int cnt = min((int)base_sel, p.k_blocks);
    for (int i = cnt + tid; i < p.k_blocks; i += kGThreads) out[(int64_t)h * p.k_blocks + i] = -1;
    if (tid == 0) p.sel_cnt[(int64_t)b * p.Hkv + h] = cnt;
    __syncthreads();                                     // base_sel has been read before the next head resets it
  }
}

}  // namespace

// Scores and selection in one launch where the keys fit its workgroups and these are all resident at once, one for
// each compute unit (two where they have nothing to wait for).  In rounds, wavefronts that have stored their scores hold
// places until their workgroup has been counted: us of one launch and of two,
//   256 workgroups: 32 heads of 1024 blocks 7.6 and 8.9, 8 heads of 4096 11.5 and 12.4; of one chunk: 5.9 and 8.0
//   512: 64 heads of 1024 13.1 and 9.9, one budget over 16 x (8 x 512) 18.8 and 14.3; of one chunk: 512 heads 9.8 and 12.0
//   1024: 256 heads of 512 24.5 and 17.1, 64 of 2048 30.0 and 19.4;  4096: 64 heads of 8192 122 and 56
// More than 256 selections of few keys are the small workgroups of select_kernel (2048 keys in registers): 1024 heads of
// 256 blocks 28 against 35 us here, 512 of 512 28.6 and 29.5, of 2048 113 and 111, of 4096 218 and 205.
Selection selection_of(const VariantParams& p) {
  const int heads = p.all_heads ? p.Hkv : 1;
  const int64_t pairs = (int64_t)heads * p.nb_max, chunks = (p.nb_max + kBlocksPerGroup - 1) / kBlocksPerGroup;
  if (heads > kMaxHeads || pairs > kManyKeys * kThreads) return kSelectFromMemory;
  if (pairs <= kKeys * kThreads && chunks * p.Hkv * p.B <= (chunks * heads == 1 ? 512 : 256)) return kSelectWithScores;
  return !p.all_heads && (int64_t)p.B * p.Hkv > 256 && p.nb_max <= 2048 ? kSelectFromMemory : kSelectFromRegisters;
}

// The scores, and with `select` (kSelectWithScores) what is kept.
hipError_t launch_retrieve(const VariantParams& p, int dtype, bool select, hipStream_t st) {
  if (dtype == SVF_F32) {
    if (p.summary_bf16) launch_d<float, __hip_bfloat16>(p, select, st);
    else launch_d<float, float>(p, select, st);
  } else {
    if (p.summary_bf16) launch_d<__hip_bfloat16, __hip_bfloat16>(p, select, st);
    else launch_d<__hip_bfloat16, float>(p, select, st);
  }
  return hipGetLastError();
}

hipError_t launch_select_kept(const VariantParams& p, hipStream_t st) {
  const int heads = p.all_heads ? p.Hkv : 1;
  const dim3 grid(1, p.Hkv / heads, p.B);
  if ((int64_t)heads * p.nb_max <= kKeys * kThreads)       // (types and rule are the scores')
    hipLaunchKernelGGL((retrieve_kernel<float, float, 64, kMeanQuery, kSelectionOnly, kKeys>), grid, dim3(kThreads), 0, st, p);
  else hipLaunchKernelGGL((retrieve_kernel<float, float, 64, kMeanQuery, kSelectionOnly, kManyKeys>), grid, dim3(kThreads), 0, st, p);
  return hipGetLastError();
}

hipError_t launch_select_global(const VariantParams& p, hipStream_t st) {
  hipLaunchKernelGGL(select_global_kernel, dim3(p.B), dim3(kGThreads), 0, st, p);
  return hipGetLastError();
}

}  // namespace svf
