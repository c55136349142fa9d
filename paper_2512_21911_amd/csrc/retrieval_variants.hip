// Retrieval variants: the block scores and the kept blocks with one rule of Sec. 3.1 exchanged.
//
//   scores:  the first draft token's score of every block PER QUERY HEAD, against the mean key
//            (Eq. 5) or against the per-channel minimum / maximum of the block's keys (Quest's
//            summary, which Sec. 3.1 starts from:  sum_c max(q_c min_c, q_c max_c) >= q . k for
//            every key of the block); the query heads of a KV head are combined by their mean or
//            their maximum.  Summaries are fp32 or bf16.  Same lane mapping as the main scores
//            kernel (eight lanes own a block, 16 channels each, fixed order of the arithmetic);
//            HBM-bound on the summaries, which are read once whatever the number of query heads.
//   select:  top-N over all (KV head, block) pairs of a sequence (Eq. 6 counts its budget over
//            the H KV heads): one workgroup per sequence; radix select over the Hkv * nb keys in
//            (head, block) order, then one ordered compaction.  Latency-bound: the keys stay in
//            registers (up to 32 per thread), one barrier per radix digit, three for the compaction.
#include <hip/hip_bf16.h>

#include "svf_device.h"

namespace svf {

namespace {

constexpr int kThreads = 256;
constexpr int kPasses = 4;             // blocks per lane group
constexpr int kHeadsPerRound = 8;      // query heads staged in LDS at a time

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

// grid: (ceil(nb_max / (kPasses * blocks per pass)), Hkv, B)
template <typename QT, typename RT, int D, bool MINMAX, bool GMAX>
__global__ __launch_bounds__(kThreads) void variant_scores_kernel(VariantParams p) {
  constexpr int LPB = kScoreLanes;
  constexpr int NCH = D / (4 * LPB);
  constexpr int BPW = kThreads / LPB;
  constexpr int ROWS = MINMAX ? 2 : 1;
  __shared__ __attribute__((aligned(16))) float qs[kHeadsPerRound][D];

  const int b = blockIdx.z, h = blockIdx.y;
  const int G = p.Hq / p.Hkv;
  const int tid = threadIdx.x, sub = tid % LPB;
  float4 r[kPasses][ROWS][NCH];
  int jj[kPasses];
#pragma unroll
  for (int u = 0; u < kPasses; ++u) {
    const int j = (blockIdx.x * kPasses + u) * BPW + tid / LPB;
    jj[u] = j;
    const int jc = j < p.nb_max ? j : p.nb_max - 1;
    const RT* row = static_cast<const RT*>(p.summaries) + ((((int64_t)b * p.Hkv + h) * p.nb_max + jc) * ROWS) * D + sub * 4;
#pragma unroll
    for (int w = 0; w < ROWS; ++w)
#pragma unroll
      for (int i = 0; i < NCH; ++i) r[u][w][i] = load4(row + w * D + i * 4 * LPB);
  }
  const int L = clamped_len(p.seq_lens, b, p.max_seq_len);
  const int nb = (L + p.block_size - 1) / p.block_size;

  float acc[kPasses];
#pragma unroll
  for (int u = 0; u < kPasses; ++u) acc[u] = GMAX ? -__builtin_inff() : 0.f;
  const QT* q0 = static_cast<const QT*>(p.q) + ((int64_t)b * p.gamma * p.Hq + (int64_t)h * G) * D;
  for (int g0 = 0; g0 < G; g0 += kHeadsPerRound) {
    const int ng = min(kHeadsPerRound, G - g0);
    if (g0 > 0) __syncthreads();                          // the round before has been read
    for (int idx = tid; idx < ng * D; idx += kThreads) (&qs[0][0])[idx] = query_value(q0[(int64_t)g0 * D + idx]);
    __syncthreads();
    for (int g = 0; g < ng; ++g) {
      float4 qv[NCH];
#pragma unroll
      for (int i = 0; i < NCH; ++i) qv[i] = *reinterpret_cast<const float4*>(&qs[g][sub * 4 + i * 4 * LPB]);
#pragma unroll
      for (int u = 0; u < kPasses; ++u) {
        float s;
        if constexpr (MINMAX) s = bound_score<NCH>(r[u][0], r[u][1], qv);
        else s = block_score<NCH>(r[u][0], qv);
        acc[u] = GMAX ? fmaxf(acc[u], s) : acc[u] + s;
      }
    }
  }
#pragma unroll
  for (int u = 0; u < kPasses; ++u) {
    const float v = GMAX ? acc[u] : acc[u] / (float)G;
    if (sub == 0 && jj[u] < p.nb_max)
      p.scores[((int64_t)b * p.Hkv + h) * p.nb_max + jj[u]] = jj[u] < nb ? v + 0.0f : 0.0f;
  }
}

template <typename QT, typename RT, int D>
void launch_scores_for(const VariantParams& p, dim3 grid, hipStream_t st) {
  if (p.minmax) {
    if (p.group_max) hipLaunchKernelGGL((variant_scores_kernel<QT, RT, D, true, true>), grid, dim3(kThreads), 0, st, p);
    else hipLaunchKernelGGL((variant_scores_kernel<QT, RT, D, true, false>), grid, dim3(kThreads), 0, st, p);
  } else {
    if (p.group_max) hipLaunchKernelGGL((variant_scores_kernel<QT, RT, D, false, true>), grid, dim3(kThreads), 0, st, p);
    else hipLaunchKernelGGL((variant_scores_kernel<QT, RT, D, false, false>), grid, dim3(kThreads), 0, st, p);
  }
}
template <typename QT, typename RT>
void launch_scores_d(const VariantParams& p, dim3 grid, hipStream_t st) {
  if (p.d == 64) launch_scores_for<QT, RT, 64>(p, grid, st);
  else launch_scores_for<QT, RT, 128>(p, grid, st);
}

// ---- top-N over the (KV head, block) pairs of a sequence ---------------------------------------
constexpr int kGThreads = 1024;
constexpr int kGWaves = kGThreads / 64;
constexpr int kMaxRegHeads = 256;      // KV heads of the kernel below

// The (head, block) pairs of a sequence in order: pair i = h * nb + j.  Thread t holds the keys of pairs
// t, t + 1024, ...: KPT of them, Hkv * nb <= 1024 KPT, Hkv <= kMaxRegHeads.  Equal keys: the lower pair wins.
//   digit  histogram in LDS (each digit its own, all zeroed up front); one barrier; every wavefront
//          scans the 256 bins for itself.  The top digits of scores are alike (same sign and most of
//          the exponent), and a wavefront's adds to one bin go one lane at a time: the lanes that
//          share the first lane's bin are counted with one add.
//   place  per 64 pairs the number of larger and of equal keys, one scan over them; a pair's rank
//          among the kept ones is then known, and with it, at the pairs that begin a head, where
//          that head's list starts.
// Four sequences, 8 heads of 512 blocks: 8.7 us (19.5 us with plain adds and a sweep of three barriers per head).
// grid: (B)
template <int KPT>
__global__ __launch_bounds__(kGThreads) void select_global_reg_kernel(VariantParams p) {
  __shared__ __attribute__((aligned(16))) uint32_t hist[4][256];
  __shared__ uint32_t seg[KPT * kGWaves];                // larger keys (low half) and equal keys of a wavefront's 64 pairs
  __shared__ uint32_t head_rank[kMaxRegHeads + 1];       // kept pairs in front of a head's first

  const int b = blockIdx.x;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int L = clamped_len(p.seq_lens, b, p.max_seq_len);
  const int nb = (L + p.block_size - 1) / p.block_size;
  const int N = p.Hkv * nb;
  const uint32_t keep_n = (uint32_t)min(N, p.n_total);
  const float* sc = p.scores + (int64_t)b * p.Hkv * p.nb_max;
  int32_t* out = p.sel_idx + (int64_t)b * p.Hkv * p.k_blocks;

  // pair t + 1024 u as (head, block), u = 0, 1, ... (nb > 0)
  struct Pair {
    int h, j, nb, dh, dj;
    __device__ Pair(int t, int nb_) : nb(nb_), dh(kGThreads / nb_), dj(kGThreads % nb_) { h = t / nb; j = t - h * nb; }
    __device__ void next() {
      h += dh;
      j += dj;
      if (j >= nb) { j -= nb; ++h; }
    }
  };
  (&hist[0][0])[tid] = 0;
  uint32_t key[KPT];
  if (nb > 0) {
    Pair at(tid, nb);
#pragma unroll
    for (int u = 0; u < KPT; ++u) {
      float v = 0.f;
      if (tid + u * kGThreads < N) v = sc[(int64_t)at.h * p.nb_max + at.j];
      key[u] = (at.j < p.n_sink || at.j >= nb - p.n_local) ? 0xffffffffu : score_key(v);
      at.next();
    }
  }
  __syncthreads();

  // key of the keep_n-th largest pair, and how many pairs equal to it are kept
  uint32_t prefix = 0, need = keep_n;
#pragma unroll
  for (int pass = 0; pass < 4; ++pass) {
    const int shift = 24 - 8 * pass;
    const uint32_t hi_mask = pass == 0 ? 0u : (0xffffffffu << (shift + 8));
#pragma unroll
    for (int u = 0; u < KPT; ++u) {
      const bool in = tid + u * kGThreads < N && (key[u] & hi_mask) == prefix;
      const uint32_t bin = (key[u] >> shift) & 0xffu;
      const uint64_t m = __ballot(in);
      if (m == 0) continue;                              // (uniform)
      const int first = __builtin_ctzll(m);
      const uint32_t bin0 = (uint32_t)__builtin_amdgcn_readlane((int)bin, first);
      const uint64_t same = __ballot(in && bin == bin0);
      if (lane == first) atomicAdd(&hist[pass][bin0], (uint32_t)__popcll(same));
      else if (in && bin != bin0) atomicAdd(&hist[pass][bin], 1u);
    }
    __syncthreads();
    // lane l owns bins 255 - 4l (in .w) down to 252 - 4l (in .x): higher bins in lower lanes
    const uint4 hq = *reinterpret_cast<const uint4*>(&hist[pass][252 - 4 * lane]);
    const uint32_t own = hq.x + hq.y + hq.z + hq.w;
    const uint32_t incl = wave_inclusive_sum(own);
    uint32_t run = incl - own;
    const uint64_t cross = __ballot(incl >= need && run < need);       // one lane (none where nothing is kept)
    if (cross == 0) break;
    uint32_t bin = 255u - 4u * (uint32_t)lane, in_bin = hq.w;
    if (run + hq.w < need) {
      run += hq.w; --bin; in_bin = hq.z;
      if (run + hq.z < need) {
        run += hq.z; --bin; in_bin = hq.y;
        if (run + hq.y < need) { run += hq.y; --bin; in_bin = hq.x; }
      }
    }
    const int src = __builtin_ctzll(cross);
    prefix |= (uint32_t)__builtin_amdgcn_readlane((int)bin, src) << shift;
    need -= (uint32_t)__builtin_amdgcn_readlane((int)run, src);
    // every key of that bin is wanted: the threshold is the smallest key of the bin, all at or above it are kept
    if (need == (uint32_t)__builtin_amdgcn_readlane((int)in_bin, src)) {
      need = 0xffffffffu;
      break;
    }
  }
  const uint32_t tau = prefix;

  const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
  for (int u = 0; u < KPT; ++u) {
    const bool in = keep_n > 0 && tid + u * kGThreads < N;
    const uint64_t gt = __ballot(in && key[u] > tau), eq = __ballot(in && key[u] == tau);
    if (lane == 0) seg[u * kGWaves + wave] = (uint32_t)__popcll(gt) | ((uint32_t)__popcll(eq) << 16);
  }
  __syncthreads();
  // (neither sum reaches 2^16: at most 32 x 1024 pairs)
  if (wave == 0) {
    constexpr int PER = (KPT * kGWaves + 63) / 64;
    uint32_t c[PER], sum = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      c[i] = lane * PER + i < KPT * kGWaves ? seg[lane * PER + i] : 0u;
      sum += c[i];
    }
    uint32_t before = wave_inclusive_sum(sum) - sum;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      if (lane * PER + i < KPT * kGWaves) seg[lane * PER + i] = before;
      before += c[i];
    }
  }
  if (tid <= p.Hkv) head_rank[tid] = keep_n;             // heads behind the last pair (an empty sequence: all)
  __syncthreads();
  uint32_t rank[KPT];                                    // kept pairs in front
#pragma unroll
  for (int u = 0; u < KPT; ++u) {
    const bool in = keep_n > 0 && tid + u * kGThreads < N;
    const uint64_t gt = __ballot(in && key[u] > tau), eq = __ballot(in && key[u] == tau);
    const uint32_t s = seg[u * kGWaves + wave];
    const uint32_t eq_before = (s >> 16) + (uint32_t)__popcll(eq & below);
    rank[u] = (s & 0xffffu) + (uint32_t)__popcll(gt & below) + min(eq_before, need);
    const bool keep = in && (key[u] > tau || (key[u] == tau && eq_before < need));
    key[u] = keep ? 1u : 0u;
  }
  if (nb > 0) {
    Pair at(tid, nb);
#pragma unroll
    for (int u = 0; u < KPT; ++u) {
      if (at.j == 0 && tid + u * kGThreads < N) head_rank[at.h] = rank[u];
      at.next();
    }
  }
  __syncthreads();
  if (nb > 0) {
    Pair at(tid, nb);
#pragma unroll
    for (int u = 0; u < KPT; ++u) {
      if (key[u]) {
        const uint32_t pos = rank[u] - head_rank[at.h];
        if (pos < (uint32_t)p.k_blocks) out[(int64_t)at.h * p.k_blocks + pos] = at.j;
      }
      at.next();
    }
  }
  for (int h = wave; h < p.Hkv; h += kGWaves) {
    const int cnt = min((int)(head_rank[h + 1] - head_rank[h]), p.k_blocks);
    for (int i = cnt + lane; i < p.k_blocks; i += 64) out[(int64_t)h * p.k_blocks + i] = -1;
    if (lane == 0) p.sel_cnt[(int64_t)b * p.Hkv + h] = cnt;
  }
}

// The same for any number of pairs: the scores are read again in every pass.
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

hipError_t launch_variant_scores(const VariantParams& p, int dtype, hipStream_t st) {
  const int bpw = kPasses * (kThreads / kScoreLanes);
  dim3 grid((p.nb_max + bpw - 1) / bpw, p.Hkv, p.B);
  if (dtype == SVF_F32) {
    if (p.summary_bf16) launch_scores_d<float, __hip_bfloat16>(p, grid, st);
    else launch_scores_d<float, float>(p, grid, st);
  } else {
    if (p.summary_bf16) launch_scores_d<__hip_bfloat16, __hip_bfloat16>(p, grid, st);
    else launch_scores_d<__hip_bfloat16, float>(p, grid, st);
  }
  return hipGetLastError();
}

hipError_t launch_select_global(const VariantParams& p, hipStream_t st) {
  // pairs of the longest possible sequence, per thread
  const int64_t per = ((int64_t)p.Hkv * p.nb_max + kGThreads - 1) / kGThreads;
  if (p.Hkv > kMaxRegHeads || per > 32) hipLaunchKernelGGL(select_global_kernel, dim3(p.B), dim3(kGThreads), 0, st, p);
  else if (per <= 4) hipLaunchKernelGGL(select_global_reg_kernel<4>, dim3(p.B), dim3(kGThreads), 0, st, p);
  else if (per <= 8) hipLaunchKernelGGL(select_global_reg_kernel<8>, dim3(p.B), dim3(kGThreads), 0, st, p);
  else hipLaunchKernelGGL(select_global_reg_kernel<32>, dim3(p.B), dim3(kGThreads), 0, st, p);
  return hipGetLastError();
}

}  // namespace svf
