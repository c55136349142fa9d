// Verification attention in fp32 arithmetic (Sec. 3.1 / 3.3: the draft queries attend to the
// retrieved blocks of their KV head and, through the draft mask, to each other).
//
// Used for fp32 inputs, and for bf16 with block or page sizes the bf16 matrix-core kernel does not
// cover (its inputs are then widened as they are loaded).
//
// Shape of the work.  The M = gamma x G query rows of a (sequence, KV head) are packed, 32 rows per
// workgroup; tokens come in tiles of 16 (draft tiles first).  A wavefront takes one tile and sixteen
// rows at a time and needs nobody else for it: both products run on the fp32 matrix instructions in
// transposed form,
//   S^T[token][row] = K[token][:] . Q[row][:]           A = K,   B = Q
//   O^T[dim][row]  += V^T[dim][token] P^T[token][row]   A = V^T, B = P
// and the k-slots of every instruction are assigned so that a lane's operands are whole 16-byte
// pieces as they lie in memory (K, Q: channels 16 j + 4 g .. + 3; V: four consecutive channels of a
// token) and the weights a lane computes are the very B operand it needs: nothing goes through LDS
// and there is no barrier before the end.  (The arithmetic rate is that of the vector ALU; what this
// replaces is every thread reading whole query and key rows out of LDS, 2 - 4 us per 32 tokens.)
//
// What bounds it.  These launches are small (fp32 is for small models and correctness runs): a
// chain of memory round trips - arguments, block ids, page table, keys - and then at most a few tiles
// of 0.43 us (d = 64) or 0.85 us (d = 128) per SIMD.  So block ids are requested before the pair's count is
// known, the eight wavefronts of a workgroup share the tiles and combine through LDS, and the splits'
// partials are merged by the workgroup that arrives last, eight splits in one trip.
// On anchor layers (SELECT) every workgroup first retrieves for its (sequence, KV head): scores of
// all its blocks with the arithmetic of the stand-alone kernel (same bits), then the top-N rule, where
// that is faster than two launches for it (f32_retrieves).
// us per anchor / reuse call, against a kernel that staged tiles in LDS for the vector ALU, with a merge
// launch behind it and two retrieval launches in front: 1024 tokens, 8 query heads of 64, 4 drafts 19.7 / 11.6
// -> 10.0 / 7.7; 6160 tokens, 4 heads of 128, 8 drafts 21.9 / 13.4 -> 13.5 / 8.9; four sequences of 32k, 32 heads of
// 128, 8 drafts 66.2 / 52.9 -> 41.1 / 31.5; bf16 in blocks of 66 (4 sequences, 32 heads, 5 drafts, 24 blocks)
// 51.4 / 41.3 -> 28.1 / 24.4.
#include <hip/hip_bf16.h>
#include <math.h>

#include "svf_device.h"
#include "svf_select.h"

namespace svf {

namespace {

constexpr int kThreads = kSelectThreads;
constexpr int kWaves = kSelectWaves;
constexpr int kRows = 32;      // query rows per workgroup
constexpr int kHalf = 16;      // query rows per wavefront
constexpr int kTile = 16;      // tokens per tile
constexpr int kScoreBatch = 8;       // passes of 64 blocks whose representatives are in flight at once
constexpr int kTableEntries = 2048;  // page-table entries kept in LDS by a retrieving workgroup

typedef float floatx4 __attribute__((ext_vector_type(4)));

// four consecutive channels (16 or 8 bytes, aligned: rows start at multiples of 16 bytes)
__device__ __forceinline__ floatx4 load4(const float* src) { return *reinterpret_cast<const floatx4*>(src); }
__device__ __forceinline__ floatx4 load4(const __hip_bfloat16* src) {
  const uint2 u = *reinterpret_cast<const uint2*>(src);
  return floatx4{__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16),
                 __uint_as_float(u.y & 0xffff0000u)};
}
__device__ __forceinline__ void store4(float* dst, floatx4 v) { *reinterpret_cast<floatx4*>(dst) = v; }
__device__ __forceinline__ void store4(__hip_bfloat16* dst, floatx4 v) {
#pragma unroll
  for (int e = 0; e < 4; ++e) dst[e] = __float2bfloat16(v[e]);   // round to nearest even
}

// Maximum / sum over the four lane groups that hold a query row (lanes l, l ^ 16, l ^ 32, l ^ 48).
__device__ __forceinline__ float row_max(float x) {
  x = fmaxf(x, __shfl_xor(x, 16, 64));
  return fmaxf(x, __shfl_xor(x, 32, 64));
}
__device__ __forceinline__ float row_sum(float x) {
  x += __shfl_xor(x, 16, 64);
  return x + __shfl_xor(x, 32, 64);
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Partials are exchanged between workgroups: device-scope accesses, which need no write-back of the
// L2 and no invalidation of the L1, only the stores' acknowledgement.
__device__ __forceinline__ void store_shared16(void* p, floatx4 v) {
  // (the store reads its registers one cycle longer than the compiler knows)
  asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" : : "v"(p), "v"(v) : "memory");
}
__device__ __forceinline__ void store_shared8(void* p, float a, float b) {
  __hip_atomic_store(static_cast<uint64_t*>(p), (uint64_t)__float_as_uint(a) | ((uint64_t)__float_as_uint(b) << 32), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t load_shared8(const void* p) {
  return __hip_atomic_load(static_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Eight 16-byte pieces `step` bytes apart, all in flight at once; n (>= 1) of them exist, the others repeat the
// first.
__device__ __forceinline__ void load_shared16x8(floatx4 (&v)[8], const char* p, int64_t step, int n) {
  const char* at[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) at[u] = p + (u < n ? u * step : 0);
  asm volatile(
      "global_load_dwordx4 %0, %8, off sc1\n\tglobal_load_dwordx4 %1, %9, off sc1\n\t"
      "global_load_dwordx4 %2, %10, off sc1\n\tglobal_load_dwordx4 %3, %11, off sc1\n\t"
      "global_load_dwordx4 %4, %12, off sc1\n\tglobal_load_dwordx4 %5, %13, off sc1\n\t"
      "global_load_dwordx4 %6, %14, off sc1\n\tglobal_load_dwordx4 %7, %15, off sc1\n\ts_waitcnt vmcnt(0)"
      : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
      : "v"(at[0]), "v"(at[1]), "v"(at[2]), "v"(at[3]), "v"(at[4]), "v"(at[5]), "v"(at[6]), "v"(at[7])
      : "memory");
}
__device__ __forceinline__ float lo_of(uint64_t w) { return __uint_as_float((uint32_t)w); }
__device__ __forceinline__ float hi_of(uint64_t w) { return __uint_as_float((uint32_t)(w >> 32)); }

template <typename T>
__device__ __forceinline__ void write_row(const AttnParams& p, int b, int h, int row, int c, floatx4 o, float m, float l) {
  const int i = row / p.G, j = h * p.G + (row - i * p.G);
  const int64_t orow = ((int64_t)b * p.gamma + i) * p.Hq + j;
  // a row that saw no key at all (no kept block, a draft mask without its own bit): zero, lse = -inf
  floatx4 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = l > 0.f ? o[e] / l : 0.f;
  store4(static_cast<T*>(p.out) + orow * p.d + c, v);
  if (p.lse && c == 0) p.lse[orow] = (m + log2f(l)) * 0.6931471805599453f;
}

// One split's (maximum, denominator) of row pr of the partials.
__device__ __forceinline__ uint64_t* part_ml(const AttnParams& p, int64_t pr) {
  return reinterpret_cast<uint64_t*>(p.part_m) + pr;
}

// Channels c .. c + 3 of a row summed over the splits, in ascending order, eight splits per trip to memory.
// A row is held by a group of eight lanes or more; its lane i (mod 8) forms the weight of split i of a trip.
struct MergedChunk {
  floatx4 o;
  float m, l;
};
__device__ __forceinline__ MergedChunk merge_chunk(const AttnParams& p, int64_t first, int c, int lane) {
  const int S = p.n_splits;
  MergedChunk r = {floatx4{0.f, 0.f, 0.f, 0.f}, -INFINITY, 0.f};
  for (int s0 = 0; s0 < S; s0 += 8) {
    const int mine = s0 + (lane & 7);
    const uint64_t ml = load_shared8(part_ml(p, first + (int64_t)min(mine, S - 1) * p.Mpad));
    floatx4 v[8];
    load_shared16x8(v, reinterpret_cast<const char*>(p.part_o + ((first + (int64_t)s0 * p.Mpad) * p.d + c)), (int64_t)p.Mpad * p.d * 4, S - s0);
    float m = mine < S ? lo_of(ml) : -INFINITY;
#pragma unroll
    for (int x = 1; x < 8; x <<= 1) m = fmaxf(m, __shfl_xor(m, x, 64));
    m = fmaxf(m, r.m);
    const float use = m == -INFINITY ? 0.f : m;
    const float alpha = fast_exp2(r.m - use);
    r.o *= alpha;
    r.l *= alpha;
    r.m = m;
    const float own = mine < S ? fast_exp2(lo_of(ml) - use) : 0.f;        // (a split that saw no token: exp2(-inf) = 0)
    const float own_l = mine < S ? own * hi_of(ml) : 0.f;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      r.l += __shfl(own_l, (lane & ~7) + u, 64);
      r.o += __shfl(own, (lane & ~7) + u, 64) * v[u];
    }
  }
  return r;
}

// grid: (n_splits, Hkv, B * row_groups)
// SELECT: see f32_retrieves; kByWavefronts: up to kWaveSelectBlocks blocks.
constexpr int kNoSelection = 0, kByWorkgroup = 1, kByWavefronts = 2;
template <typename T, int D, int SELECT>
__global__ __launch_bounds__(kThreads) void verify_attn_f32_kernel(AttnParams p, int row_groups) {
  constexpr int NJ = D / 16;                  // 16-channel steps of the first product
  constexpr int NH = D / 64;                  // four-channel pieces of a V row per lane
  constexpr int kPitch = D + 4;               // floats per parked row
  constexpr int NCH = D / (4 * kScoreLanes);  // four-channel pieces of a representative per lane
  constexpr int kSelectBytes = SELECT == kByWavefronts ? sizeof(WaveSelectScratch) : sizeof(SelectScratch);
  constexpr int kRetrievalBytes = (D + kMaxSelectBlocks + kTableEntries) * 4 + kSelectBytes;
  constexpr int kParkedBytes = kWaves * kHalf * kPitch * 4;
  __shared__ __attribute__((aligned(16))) unsigned char smem[SELECT && kRetrievalBytes > kParkedBytes ? kRetrievalBytes : kParkedBytes];
  __shared__ float s_m[kWaves][kHalf], s_l[kWaves][kHalf];
  __shared__ int32_t s_sel[SELECT ? kMaxSelectBlocks : 1];
  __shared__ int s_last;
  // the argument block is read piecemeal below: touch each of its lines once now
  {
    const __attribute__((address_space(4))) uint32_t* ka =
        (const __attribute__((address_space(4))) uint32_t*)__builtin_amdgcn_kernarg_segment_ptr();
    static_assert(sizeof(AttnParams) > 5 * 64, "argument block shorter than the lines touched");
    const uint32_t w0 = ka[0], w1 = ka[16], w2 = ka[32], w3 = ka[48], w4 = ka[64], w5 = ka[80];
    asm volatile("" : : "s"(w0), "s"(w1), "s"(w2), "s"(w3), "s"(w4), "s"(w5));
  }
  const int split = blockIdx.x, h = blockIdx.y;
  const int b = blockIdx.z / row_groups, rg = blockIdx.z - b * row_groups;
  const int pair = b * p.Hkv + h;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int l16 = lane & 15, g = lane >> 4, slot = lane & 15;
  // rows: one half of sixteen or two; the wavefronts of a half share the tiles
  const int halves = p.M - rg * kRows > kHalf ? 2 : 1;
  const int teams = kWaves / halves;
  const int half = halves == 2 ? wave & 1 : 0, team = halves == 2 ? wave >> 1 : wave;
  const int row = rg * kRows + half * kHalf + l16;
  const bool row_ok = row < p.M;
  const int di = row_ok ? row / p.G : 0;      // draft index of this lane's row
  const int hq = h * p.G + (row_ok ? row - di * p.G : 0);
  const int32_t* const table_row = p.table + (int64_t)b * p.kv.max_pages;
  int32_t* const s_table = reinterpret_cast<int32_t*>(smem + (D + kMaxSelectBlocks) * 4 + kSelectBytes);
  const bool table_in_lds = SELECT && p.kv.page_size != 0 && p.kv.max_pages <= kTableEntries;

  const int tiles_d = (p.gamma + kTile - 1) / kTile;
  const int step = teams * p.n_splits;
  const int t_first = split + p.n_splits * team;             // (the splits' wavefronts fill up evenly)

  // ---- everything whose address is known is requested now ----
  QueryHeads<T> heads;
  const T* const q0 = static_cast<const T*>(p.q) + ((int64_t)b * p.gamma * p.Hq + (int64_t)h * p.G) * D + (tid & (D - 1));
  floatx4 reps[SELECT ? kScoreBatch : 1][NCH];
  const float* const reps_lane = SELECT ? p.reps + (int64_t)pair * p.nb_max * D + (tid % kScoreLanes) * 4 : nullptr;
  auto load_reps = [&](int first) {
#pragma unroll
    for (int u = 0; u < kScoreBatch; ++u)
      if ((first + u) * 64 < p.nb_max) {
        const float* r = reps_lane + (int64_t)min((first + u) * 64 + tid / kScoreLanes, p.nb_max - 1) * D;
#pragma unroll
        for (int i = 0; i < NCH; ++i) reps[SELECT ? u : 0][i] = load4(r + i * 4 * kScoreLanes);
      }
  };
  int table_own[kTableEntries / kThreads];
  if constexpr (SELECT) {
    if (tid < D) heads = load_query_heads<T>(q0, p.G, D);
    load_reps(0);
    if (table_in_lds) {
#pragma unroll
      for (int u = 0; u < kTableEntries / kThreads; ++u)
        if (u * kThreads < p.kv.max_pages) table_own[u] = table_row[min(tid + u * kThreads, p.kv.max_pages - 1)];
    }
  }
  const int L = clamped_len(p.seq_lens, b, p.max_seq_len);
  int cnt = 0;
  if constexpr (!SELECT) cnt = p.sel_cnt[pair];
  const int32_t* const sel_g = p.sel_idx + (int64_t)pair * p.k_blocks;
  // block of this lane's slot of cache tile t (a clamped index where there is none)
  auto block_index = [&](int t) {
    const int s = (t - tiles_d) * kTile + slot;
    return p.block_shift >= 0 ? s >> p.block_shift : s / p.block_size;
  };
  auto load_block = [&](int t) -> int {
    if (t < tiles_d) return -1;
    const int i = min(block_index(t), p.k_blocks - 1);
    if constexpr (SELECT) return s_sel[min(i, kMaxSelectBlocks - 1)];
    else return sel_g[i];
  };
  int blk = -1;
  if constexpr (!SELECT) blk = load_block(t_first);
  uint64_t mask = 0;
  if (row_ok) {
    if (p.draft_mask) mask = p.draft_mask[p.mask_per_batch ? (int64_t)b * p.gamma + di : di];
    else mask = di >= 63 ? ~0ull : ((2ull << di) - 1ull);
  }
  floatx4 q[NJ];
  {
    const T* src = static_cast<const T*>(p.q) + (((int64_t)b * p.gamma + di) * p.Hq + hq) * D + 4 * g;
#pragma unroll
    for (int j = 0; j < NJ; ++j) q[j] = load4(src + 16 * j);
  }

  // ---- retrieval ----
  if constexpr (SELECT) {
    float* const s_q0 = reinterpret_cast<float*>(smem);
    uint32_t* const s_keys = reinterpret_cast<uint32_t*>(smem + D * 4);
    SelectScratch* const sc = reinterpret_cast<SelectScratch*>(smem + (D + kMaxSelectBlocks) * 4);
    WaveSelectScratch* const wsc = reinterpret_cast<WaveSelectScratch*>(sc);
    if constexpr (SELECT == kByWavefronts) clear_counts(wsc, tid);
    else
      for (int i = tid; i < 4 * 256; i += kThreads) (&sc->hist[0][0])[i] = 0;
    if (tid < D) s_q0[tid] = mean_query_channel<T>(heads, q0, p.G, D);
    __syncthreads();
    const int nb = (L + p.block_size - 1) / p.block_size;
    cnt = min(p.k_blocks, nb);
    const int sub = tid % kScoreLanes;
    float4 qv[NCH];
#pragma unroll
    for (int i = 0; i < NCH; ++i) qv[i] = *reinterpret_cast<const float4*>(s_q0 + sub * 4 + i * 4 * kScoreLanes);
    for (int first = 0; first * 64 < nb; first += kScoreBatch) {
      if (first > 0) load_reps(first);
#pragma unroll
      for (int u = 0; u < kScoreBatch; ++u) {
        if ((first + u) * 64 >= nb) continue;               // (uniform)
        float4 r[NCH];
#pragma unroll
        for (int i = 0; i < NCH; ++i) r[i] = make_float4(reps[u][i][0], reps[u][i][1], reps[u][i][2], reps[u][i][3]);
        const float v = block_score<NCH>(r, qv);
        const int j = (first + u) * 64 + tid / kScoreLanes;
        if (sub == 0 && j < nb) {
          const uint32_t key = (j < p.n_sink || j >= nb - p.n_local) ? 0xffffffffu : score_key(v + 0.0f);
          s_keys[j] = key;
          if constexpr (SELECT == kByWavefronts) count_key(wsc, key);
          else atomicAdd(&sc->hist[0][key >> 24], 1u);
        }
      }
    }
    if (table_in_lds) {
#pragma unroll
      for (int u = 0; u < kTableEntries / kThreads; ++u)
        if (tid + u * kThreads < p.kv.max_pages) s_table[tid + u * kThreads] = table_own[u];
    }
    __syncthreads();
    if constexpr (SELECT == kByWavefronts) {
      if (cnt > 0) wave_select(s_keys, wsc, nb, cnt, s_sel, lane);
    } else {
      if (cnt > 0) workgroup_select(s_keys, sc, nb, cnt, s_sel, tid, lane, wave, true);
      __syncthreads();
    }
    if (split == 0 && rg == 0) {
      for (int i = tid; i < p.k_blocks; i += kThreads) p.sel_idx_out[(int64_t)pair * p.k_blocks + i] = i < cnt ? s_sel[i] : -1;
      if (tid == 0) p.sel_cnt_out[pair] = cnt;
    }
    blk = load_block(t_first);
  } else {
    cnt = min(max(cnt, 0), p.k_blocks);
  }
  const int n_prefix = cnt * p.block_size;    // token slots of the selected blocks
  const int tiles = tiles_d + (n_prefix + kTile - 1) / kTile;

  const int64_t kv_head = (int64_t)h * p.kv.stride_head;
  const int64_t draft0 = ((int64_t)b * p.gamma * p.Hkv + h) * D;

  float m_run = -INFINITY, l_run = 0.f;
  floatx4 acc[NH][4];                         // [hh][e], value v: channel 64 hh + 16 g + 4 v + e of this lane's row
#pragma unroll
  for (int hh = 0; hh < NH; ++hh)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[hh][e] = floatx4{0.f, 0.f, 0.f, 0.f};

  for (int t = t_first; t < tiles; t += step) {
    // where the tile's tokens are: lanes i, i + 16, ... resolve slot i.  A slot without a token
    // reads the first draft's row (always there) and counts nothing.
    bool here;
    const T *kp = static_cast<const T*>(p.k_draft) + draft0, *vp = static_cast<const T*>(p.v_draft) + draft0;
    if (t < tiles_d) {
      const int i = t * kTile + slot;
      here = i < p.gamma;
      const int64_t off = here ? (int64_t)i * p.Hkv * D : 0;
      kp += off;
      vp += off;
    } else {
      const int s = (t - tiles_d) * kTile + slot;
      const int tok = blk * p.block_size + (s - block_index(t) * p.block_size);
      here = s < n_prefix && blk >= 0 && tok >= 0 && tok < L;
      if (here) {
        int64_t off;
        if (p.kv.page_size == 0) {
          off = (int64_t)b * p.kv.stride_page + (int64_t)tok * p.kv.stride_tok;
        } else {
          const int pg = p.kv.page_shift >= 0 ? tok >> p.kv.page_shift : tok / p.kv.page_size;
          const int phys = table_in_lds ? s_table[pg] : table_row[pg];
          off = (int64_t)phys * p.kv.stride_page + (int64_t)(tok - pg * p.kv.page_size) * p.kv.stride_tok;
        }
        kp = static_cast<const T*>(p.K) + off + kv_head;
        vp = static_cast<const T*>(p.V) + off + kv_head;
      }
    }
    const uint32_t valid = (uint32_t)__ballot(here) & 0xffffu;
    auto lane_ptr = [&](const T* ptr, int from) {
      const uint64_t a = reinterpret_cast<uint64_t>(ptr);
      const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)a, from, 64), hi = (uint32_t)__shfl((int)(uint32_t)(a >> 32), from, 64);
      return reinterpret_cast<const T*>(((uint64_t)hi << 32) | lo);
    };
    // K: token l16, channels 16 j + 4 g .. + 3;  V: token 4 g + v, channels 64 hh + 4 l16 .. + 3
    floatx4 k[NJ], vv[4][NH];
#pragma unroll
    for (int j = 0; j < NJ; ++j) k[j] = load4(kp + 4 * g + 16 * j);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const T* src = lane_ptr(vp, 4 * g + v) + 4 * l16;
#pragma unroll
      for (int hh = 0; hh < NH; ++hh) vv[v][hh] = load4(src + 64 * hh);
    }
    if (t + step < tiles) blk = load_block(t + step);       // for the next tile

    floatx4 s2[2] = {floatx4{0.f, 0.f, 0.f, 0.f}, floatx4{0.f, 0.f, 0.f, 0.f}};   // (two chains of matrix instructions)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) s2[e & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(k[j][e], q[j][e], s2[e & 1], 0, 0, 0);
    floatx4 s = s2[0] + s2[1];                              // value v: token 4 g + v
    const uint32_t allowed = t < tiles_d ? valid & (uint32_t)(mask >> (t * kTile)) : valid;
    float m_tile = -INFINITY;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const bool vis = row_ok && ((allowed >> (4 * g + v)) & 1u);
      s[v] = vis ? s[v] * p.scale_log2 : -INFINITY;
      m_tile = fmaxf(m_tile, s[v]);
    }
    const float m_new = fmaxf(m_run, row_max(m_tile));
    const float m_use = m_new == -INFINITY ? 0.f : m_new;
    const float alpha = fast_exp2(m_run - m_use);           // m_run = -inf gives 0
    m_run = m_new;
    l_run *= alpha;
#pragma unroll
    for (int hh = 0; hh < NH; ++hh)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[hh][e] *= alpha;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float pe = fast_exp2(s[v] - m_use);
      l_run += pe;
      const bool real = (valid >> (4 * g + v)) & 1u;        // (zero times what stands there might be NaN)
#pragma unroll
      for (int hh = 0; hh < NH; ++hh)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          acc[hh][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(real ? vv[v][hh][e] : 0.f, pe, acc[hh][e], 0, 0, 0);
    }
  }

  // ---- the wavefronts of a half are brought together through LDS ----
  float* const parked = reinterpret_cast<float*>(smem);     // [wavefront][row][kPitch]
  l_run = row_sum(l_run);
  if (SELECT) __syncthreads();                              // (the page table has been read)
  if (g == 0) {
    s_m[wave][l16] = m_run;
    s_l[wave][l16] = l_run;
  }
#pragma unroll
  for (int hh = 0; hh < NH; ++hh)
#pragma unroll
    for (int v = 0; v < 4; ++v)
      store4(parked + (wave * kHalf + l16) * kPitch + 64 * hh + 16 * g + 4 * v,
             floatx4{acc[hh][0][v], acc[hh][1][v], acc[hh][2][v], acc[hh][3][v]});
  __syncthreads();
  const int64_t first = ((int64_t)pair * p.n_splits) * p.Mpad + rg * kRows;       // row of split 0 in the partials
  const int n_rows = min(p.M - rg * kRows, kRows);
  const int busy = min(max((tiles - split + p.n_splits - 1) / p.n_splits, 0), teams);      // teams that had a tile
  for (int i = tid; i < n_rows * (D / 4); i += kThreads) {
    const int r = i / (D / 4), c = 4 * (i & (D / 4 - 1));
    const int w0 = halves == 2 ? r >> 4 : 0, rr = r & 15;
    float m = -INFINITY, l = 0.f;
    for (int tm = 0; tm < busy; ++tm) m = fmaxf(m, s_m[w0 + tm * halves][rr]);
    const float use = m == -INFINITY ? 0.f : m;
    floatx4 o = {0.f, 0.f, 0.f, 0.f};
    for (int tm = 0; tm < busy; ++tm) {
      const int w = w0 + tm * halves;
      const float f = fast_exp2(s_m[w][rr] - use);
      l += f * s_l[w][rr];
      o += f * load4(parked + (w * kHalf + rr) * kPitch + c);
    }
    if (p.n_splits == 1) {
      write_row<T>(p, b, h, rg * kRows + r, c, o, m, l);
    } else {
      const int64_t pr = first + (int64_t)split * p.Mpad + r;
      store_shared16(p.part_o + pr * D + c, o);
      if (c == 0) store_shared8(part_ml(p, pr), m, l);
    }
  }
  if (p.n_splits == 1) return;
  // ---- the workgroup that arrives last merges the splits ----
  __builtin_amdgcn_s_waitcnt((0xf << 8) | (0x7 << 4));      // vmcnt(0): this wavefront's partials have been acknowledged
  asm volatile("" ::: "memory");
  __syncthreads();
  if (tid == 0) {
    uint64_t* const arrivals = p.tickets + ((int64_t)rg * gridDim.y * (gridDim.z / row_groups) + pair) * kTicketWords + 2;
    const uint64_t prev = __hip_atomic_fetch_add(arrivals, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_last = prev == (uint64_t)(p.n_splits - 1);
    if (s_last) __hip_atomic_store(arrivals, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (!s_last) return;
  // (whole wavefronts: lanes past the last row follow it)
  for (int i0 = wave * 64; i0 < n_rows * (D / 4); i0 += kThreads) {
    const int i = i0 + lane, r = min(i / (D / 4), n_rows - 1), cl = i & (D / 4 - 1);
    const MergedChunk x = merge_chunk(p, first + r, 4 * cl, lane);
    if (i < n_rows * (D / 4)) write_row<T>(p, b, h, rg * kRows + r, 4 * cl, x.o, x.m, x.l);
  }
}

template <typename T, int D>
hipError_t launch(const AttnParams& p, hipStream_t st) {
  const int row_groups = p.Mpad / kRows;
  const dim3 grid(p.n_splits, p.Hkv, p.B * row_groups);
  if (!p.reps) hipLaunchKernelGGL((verify_attn_f32_kernel<T, D, kNoSelection>), grid, dim3(kThreads), 0, st, p, row_groups);
  else if (p.nb_max <= kWaveSelectBlocks) hipLaunchKernelGGL((verify_attn_f32_kernel<T, D, kByWavefronts>), grid, dim3(kThreads), 0, st, p, row_groups);
  else hipLaunchKernelGGL((verify_attn_f32_kernel<T, D, kByWorkgroup>), grid, dim3(kThreads), 0, st, p, row_groups);
  return hipGetLastError();
}

// (tiles, halves) units of one (sequence, KV head, row group): what its wavefronts share out.
int64_t tiles_of(const svf_shape_t& s) {
  return ((int64_t)s.k_blocks * s.block_size + kTile - 1) / kTile + (s.gamma + kTile - 1) / kTile;
}
int64_t units_of(const svf_shape_t& s) { return tiles_of(s) * (s.gamma * (s.Hq / s.Hkv) > kHalf ? 2 : 1); }
int64_t groups_of(const svf_shape_t& s) {
  const int64_t M = (int64_t)s.gamma * (s.Hq / s.Hkv);
  return (int64_t)s.B * s.Hkv * ((M + kRows - 1) / kRows);
}

}  // namespace

// Splits per (sequence, KV head, row group).  A unit is a tile for sixteen rows; a workgroup has four SIMDs.
// Eight splits are merged in one trip to memory (2 us with the exchange), so the splits are a multiple of eight (or as
// many as there are tiles), also for few units rather than let these queue in one workgroup (or in sixteen wavefronts
// there); four units are as fast in one workgroup.  From 41 units on two trips pay, behind that the splits grow with
// the square root.  Never more than 256 workgroups: a compute unit's registers hold one at a time at d = 128, and at
// d = 64, where they hold two, a second one costs what its work saves; and where 16 splits would
// fill the 256, 8 of them twice as long are the faster ones up to 80 units.  us per call,
// d = 64 and d = 128: 9 units 7.4 / 8.4 (2 splits 8.1 / 9.2; one 9.1 / 11.1), 17 units 7.8 / 9.1 (16 splits 8.3 / 9.4),
// 66 units 8.7 / 12.8 with 16 splits, 9.0 / 13.7 with 8, 9.9 / 15.1 with 9; 130 units 10.0 / 15.3 with 16, 10.6 / 16.7 with 18;
// 258 units 12.3 / 18.7 with 24, 12.8 / 20.0 with 25; 2049 units (d = 128) 30.8 with 68, 45 with 257; 8 pairs of 1026 units
// 35.5 with 32 splits, 50.7 with 49; 32 pairs of 129 units (d = 128) 31.5 with 8, 43.9 with 16; of 258 units (d = 64)
// 18.9 with 8, 19.2 with 16; 16 pairs of 258 units (d = 64) 14.7 with 16, 18.3 with 32; 16 row groups of 72 units 9.7 / 14.7
// with 8, 10.1 / 15.5 with 16.
int f32_splits(const svf_shape_t& s) {
  const int64_t units = units_of(s), groups = groups_of(s);
  if (units <= 4) return 1;
  const int64_t tiles = tiles_of(s);
  const int64_t trips = (int64_t)(1.5 * sqrt((double)units) / 8);      // of the merge
  int64_t want = units <= 40 ? 8 : 8 * (trips > 2 ? trips : 2);
  if (want > tiles) want = tiles;
  const int64_t most = groups < 256 ? 256 / groups : 1;
  if (want > 8 && most <= 16 && units < 80) want = 8;
  return (int)(want < most ? want : most);
}

// Whether anchor layers retrieve inside the attention kernel, every workgroup for itself.  One round of
// workgroups reads a pair's representatives (512 KB at most) faster than another launch is made, also if
// all splits read the same ones.  Several rounds (256 groups and more) do that one after the other: 512
// workgroups 26.1 against 31.5 us with 32 KB each, 30.4 and 31.5 with 64 KB, 35.7 and 32.1 with 128 KB.
bool f32_retrieves(const svf_shape_t& s) {
  const int64_t nb = ((int64_t)s.max_seq_len + s.block_size - 1) / s.block_size;
  const int64_t workgroups = groups_of(s) * f32_splits(s);
  return nb <= kMaxSelectBlocks && (workgroups <= 256 || workgroups * nb * s.d * 4 <= ((int64_t)32 << 20));
}

hipError_t launch_verify_attn_f32(const AttnParams& p, int dtype, hipStream_t st) {
  if (dtype == SVF_F32) return p.d == 64 ? launch<float, 64>(p, st) : launch<float, 128>(p, st);
  return p.d == 64 ? launch<__hip_bfloat16, 64>(p, st) : launch<__hip_bfloat16, 128>(p, st);
}

}  // namespace svf
