// Verification attention, vector-ALU kernel (Sec. 3.1 / 3.3: the draft queries attend to the
// retrieved blocks of their KV head and, through the draft mask, to each other).
//
// Used for fp32 inputs and for block or page sizes the matrix-core kernel does not cover.
// Split-K over the selected tokens: workgroup (split, kv head, sequence x row group) walks
// its share of 32-token tiles (prefix tiles first, then the draft tile(s)), staging K and V
// through LDS as fp32; thread (r, sub) owns query row r of the row group and the channels
// 4 * sub .. 4 * sub + 3 of every 32.  The 8 lanes of a row compute its 32 logits, keep the
// running maximum and denominator in registers (online softmax in the log2 domain) and
// accumulate its output.  Each split writes an unnormalised partial (o, m, l); a second kernel
// merges the splits with the log-sum-exp rule and writes out / lse.
//
// A workgroup usually has one tile, so what bounds it is its memory round trips (count, block id,
// page, key) and, behind them, LDS reads: each of the 256 threads reads a whole query row and four
// key rows.  They are read 16 bytes at a time from rows of D + 4 floats (the 8 rows or tokens of a
// wavefront's read then lie in different banks), and queries, keys and values are all requested
// before anything waits.  Every sum keeps its order.
// Whole steps, against scalar LDS reads from unpadded rows and a merge of one split at a time, same bits
// in fp32: two layers of 1024 tokens (8 query heads of 64, 4 drafts, 8 blocks of 16) 37.7 -> 28.8 us;
// two sequences of 8k tokens (16 heads of 128, 8 drafts, 16 blocks of 32) 77.7 -> 39.9 us; bf16 in
// blocks of 66 (4 sequences, 32 heads, 5 drafts, 24 blocks) 229 -> 90.6 us.
#include <hip/hip_bf16.h>

#include "svf_device.h"

namespace svf {

namespace {

constexpr int kThreads = 256;
constexpr int kRows = 32;      // query rows per workgroup
constexpr int kTile = 32;      // tokens per tile
constexpr int kSub = 8;        // lanes per query row
constexpr int kPPitch = kTile + 4;   // floats per row of weights
constexpr int kMergeBatch = 16;      // splits whose partials the merge has in flight at once

// four consecutive channels (16 or 8 bytes, aligned: rows start at multiples of 16 bytes)
__device__ __forceinline__ float4 load4(const float* src) { return *reinterpret_cast<const float4*>(src); }
__device__ __forceinline__ float4 load4(const __hip_bfloat16* src) {
  const uint2 u = *reinterpret_cast<const uint2*>(src);
  return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16),
                     __uint_as_float(u.y & 0xffff0000u));
}

// grid: (n_splits, Hkv, B * row_groups)
template <typename T, int D>
__global__ __launch_bounds__(kThreads) void verify_attn_valu_kernel(AttnParams p, int row_groups) {
  constexpr int KP = D + 4;                   // padded Q and K rows (floats)
  constexpr int NC = D / (4 * kSub);          // four-channel chunks per thread: sub, sub + 8, ...
  __shared__ __attribute__((aligned(16))) float sQ[kRows * KP];
  __shared__ __attribute__((aligned(16))) float sK[kTile * KP];
  __shared__ __attribute__((aligned(16))) float sV[kTile * D];
  __shared__ __attribute__((aligned(16))) float sP[kRows * kPPitch];
  __shared__ int sTok[kTile];                 // >= 0: prefix token, -1: invalid, -2 - t: draft t

  const int split = blockIdx.x, h = blockIdx.y;
  const int b = blockIdx.z / row_groups, rg = blockIdx.z - b * row_groups;
  const int tid = threadIdx.x;
  const int r = tid / kSub, sub = tid % kSub;
  const int row = rg * kRows + r;             // row inside the (b, h) pair: draft * G + group head
  const bool row_ok = row < p.M;
  const int di = row_ok ? row / p.G : 0;      // draft index of this row
  const int hq = h * p.G + (row_ok ? row % p.G : 0);

  const int L = clamped_len(p.seq_lens, b, p.max_seq_len);
  const int cnt = min(max(p.sel_cnt[(int64_t)b * p.Hkv + h], 0), p.k_blocks);
  const int32_t* sel = p.sel_idx + ((int64_t)b * p.Hkv + h) * p.k_blocks;
  const int n_prefix = cnt * p.block_size;    // token slots of the selected blocks
  const int tiles_p = (n_prefix + kTile - 1) / kTile;
  const int tiles_d = (p.gamma + kTile - 1) / kTile;
  const int tiles = tiles_p + tiles_d;
  const int per = (tiles + p.n_splits - 1) / p.n_splits;
  const int tile0 = split * per;
  const int tile1 = min(tiles, tile0 + per);

  uint64_t mask = 0;
  if (row_ok) {
    if (p.draft_mask) mask = p.draft_mask[p.mask_per_batch ? (int64_t)b * p.gamma + di : di];
    else mask = di >= 63 ? ~0ull : ((2ull << di) - 1ull);
  }

  // this row's queries: chunks sub, sub + 8, ... (stored to LDS behind the first tile's requests)
  float4 qv[NC];
  {
    const T* qsrc = static_cast<const T*>(p.q) + (((int64_t)b * p.gamma + di) * p.Hq + hq) * D + 4 * sub;
#pragma unroll
    for (int i = 0; i < NC; ++i) qv[i] = row_ok ? load4(qsrc + 4 * kSub * i) : make_float4(0.f, 0.f, 0.f, 0.f);
  }

  float m_run = -INFINITY, l_run = 0.f;
  float4 acc[NC];
#pragma unroll
  for (int i = 0; i < NC; ++i) acc[i] = make_float4(0.f, 0.f, 0.f, 0.f);

  for (int tile = tile0; tile < tile1; ++tile) {
    // token r of the tile is loaded by the 8 threads (r, sub)
    int code = -1;
    if (tile < tiles_p) {
      const int slot = tile * kTile + r;
      if (slot < n_prefix) {
        const int bi = slot / p.block_size;
        const int blk = sel[bi];
        const int t = blk * p.block_size + (slot - bi * p.block_size);
        if (blk >= 0 && t < L) code = t;
      }
    } else {
      const int t = (tile - tiles_p) * kTile + r;
      if (t < p.gamma) code = -2 - t;
    }
    float4 kv[NC], vv[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) kv[i] = vv[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (code != -1) {
      const T *ksrc, *vsrc;
      if (code >= 0) {
        const int64_t off = token_offset(p.kv, p.table, b, code) + (int64_t)h * p.kv.stride_head + 4 * sub;
        ksrc = static_cast<const T*>(p.K) + off;
        vsrc = static_cast<const T*>(p.V) + off;
      } else {
        const int64_t off = (((int64_t)b * p.gamma + (-2 - code)) * p.Hkv + h) * D + 4 * sub;
        ksrc = static_cast<const T*>(p.k_draft) + off;
        vsrc = static_cast<const T*>(p.v_draft) + off;
      }
#pragma unroll
      for (int i = 0; i < NC; ++i) {
        kv[i] = load4(ksrc + 4 * kSub * i);
        vv[i] = load4(vsrc + 4 * kSub * i);
      }
    }
    if (tile == tile0) {
#pragma unroll
      for (int i = 0; i < NC; ++i) *reinterpret_cast<float4*>(sQ + r * KP + 4 * sub + 4 * kSub * i) = qv[i];
    } else {
      __syncthreads();                        // previous tile fully consumed
    }
    if (sub == 0) sTok[r] = code;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      *reinterpret_cast<float4*>(sK + r * KP + 4 * sub + 4 * kSub * i) = kv[i];
      *reinterpret_cast<float4*>(sV + r * D + 4 * sub + 4 * kSub * i) = vv[i];
    }
    __syncthreads();

    // logits of row r against tokens sub, sub + 8, sub + 16, sub + 24
    float s[kTile / kSub];
#pragma unroll
    for (int u = 0; u < kTile / kSub; ++u) s[u] = 0.f;
#pragma unroll 4
    for (int c = 0; c < D; c += 4) {
      const float4 a = *reinterpret_cast<const float4*>(sQ + r * KP + c);
#pragma unroll
      for (int u = 0; u < kTile / kSub; ++u) {
        const float4 k = *reinterpret_cast<const float4*>(sK + (sub + kSub * u) * KP + c);
        s[u] += a.x * k.x;
        s[u] += a.y * k.y;
        s[u] += a.z * k.z;
        s[u] += a.w * k.w;
      }
    }
    float m_tile = -INFINITY;
#pragma unroll
    for (int u = 0; u < kTile / kSub; ++u) {
      const int code_u = sTok[sub + kSub * u];
      bool vis = code_u >= 0;
      if (code_u <= -2) vis = (mask >> (-2 - code_u)) & 1ull;
      s[u] = vis && row_ok ? s[u] * p.scale_log2 : -INFINITY;
      m_tile = fmaxf(m_tile, s[u]);
    }
#pragma unroll
    for (int o = 1; o < kSub; o <<= 1) m_tile = fmaxf(m_tile, __shfl_xor(m_tile, o, 64));
    const float m_new = fmaxf(m_run, m_tile);
    const float m_use = m_new == -INFINITY ? 0.f : m_new;
    const float alpha = exp2f(m_run - m_use);          // m_run = -inf gives 0
    float l_tile = 0.f;
#pragma unroll
    for (int u = 0; u < kTile / kSub; ++u) {
      const float pe = exp2f(s[u] - m_use);
      l_tile += pe;
      sP[r * kPPitch + sub + kSub * u] = pe;
    }
#pragma unroll
    for (int o = 1; o < kSub; o <<= 1) l_tile += __shfl_xor(l_tile, o, 64);
    l_run = l_run * alpha + l_tile;
    m_run = m_new;
    __syncthreads();                          // sP complete (rows are wave-local, but keep it simple)

#pragma unroll
    for (int i = 0; i < NC; ++i) {
      acc[i].x *= alpha;
      acc[i].y *= alpha;
      acc[i].z *= alpha;
      acc[i].w *= alpha;
    }
#pragma unroll 2
    for (int t = 0; t < kTile; t += 4) {
      const float4 pe4 = *reinterpret_cast<const float4*>(sP + r * kPPitch + t);
      const float pe[4] = {pe4.x, pe4.y, pe4.z, pe4.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
#pragma unroll
        for (int i = 0; i < NC; ++i) {
          const float4 v = *reinterpret_cast<const float4*>(sV + (t + e) * D + 4 * sub + 4 * kSub * i);
          acc[i].x += pe[e] * v.x;
          acc[i].y += pe[e] * v.y;
          acc[i].z += pe[e] * v.z;
          acc[i].w += pe[e] * v.w;
        }
      }
    }
  }

  // partial result of this split
  const int64_t pr = (((int64_t)b * p.Hkv + h) * p.n_splits + split) * p.Mpad + row;
  if (row < p.Mpad) {
#pragma unroll
    for (int i = 0; i < NC; ++i) *reinterpret_cast<float4*>(p.part_o + pr * D + 4 * sub + 4 * kSub * i) = acc[i];
    if (sub == 0) {
      p.part_m[pr] = m_run;
      p.part_l[pr] = l_run;
    }
  }
}

template <typename T>
__device__ __forceinline__ void store_out(T* dst, float v);
template <>
__device__ __forceinline__ void store_out<float>(float* dst, float v) { *dst = v; }
template <>
__device__ __forceinline__ void store_out<__hip_bfloat16>(__hip_bfloat16* dst, float v) {
  *dst = __float2bfloat16(v);   // round to nearest even
}

// grid: (M, Hkv, B); block: D threads.  Merges the per-split partials of one query row.
// Memory round trips bound it (a split at a time: two per split): a wavefront finds the maximum with
// a split per lane, and the partials of kMergeBatch splits are requested together, the first ones
// before the maximum is known.  The splits are added in ascending order.
template <typename T>
__global__ void merge_splits_kernel(AttnParams p) {
  const int row = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
  const int c = threadIdx.x;
  const int D = p.d;
  const int S = p.n_splits;
  const int64_t base = ((int64_t)b * p.Hkv + h) * S;
  float bm[kMergeBatch], bl[kMergeBatch], bo[kMergeBatch];
  auto request = [&](int s0) {
#pragma unroll
    for (int u = 0; u < kMergeBatch; ++u) {
      const int64_t pr = (base + min(s0 + u, S - 1)) * p.Mpad + row;
      bm[u] = p.part_m[pr];
      bl[u] = p.part_l[pr];
      bo[u] = p.part_o[pr * D + c];
    }
  };
  request(0);
  float m = -INFINITY;
  for (int s = c & 63; s < S; s += 64) m = fmaxf(m, p.part_m[(base + s) * p.Mpad + row]);
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
  float l = 0.f, o = 0.f;
  for (int s0 = 0; s0 < S; s0 += kMergeBatch) {
    if (s0) request(s0);
#pragma unroll
    for (int u = 0; u < kMergeBatch; ++u) {
      if (s0 + u >= S || bm[u] == -INFINITY) continue;
      const float w = exp2f(bm[u] - m);
      l += w * bl[u];
      o += w * bo[u];
    }
  }
  const int i = row / p.G, j = h * p.G + row % p.G;
  const int64_t orow = ((int64_t)b * p.gamma + i) * p.Hq + j;
  // a row that saw no key at all (no kept block, a draft mask without its own bit): zero, lse = -inf
  store_out<T>(static_cast<T*>(p.out) + orow * D + c, l > 0.f ? o / l : 0.f);
  if (p.lse && c == 0) p.lse[orow] = (m + log2f(l)) * 0.6931471805599453f;
}

}  // namespace

hipError_t launch_merge_splits(const AttnParams& p, int dtype, hipStream_t st) {
  dim3 grid(p.M, p.Hkv, p.B);
  if (dtype == SVF_F32) hipLaunchKernelGGL(merge_splits_kernel<float>, grid, dim3(p.d), 0, st, p);
  else hipLaunchKernelGGL(merge_splits_kernel<__hip_bfloat16>, grid, dim3(p.d), 0, st, p);
  return hipGetLastError();
}

hipError_t launch_verify_attn_valu(const AttnParams& p, int dtype, hipStream_t st) {
  const int row_groups = p.Mpad / kRows;
  dim3 grid(p.n_splits, p.Hkv, p.B * row_groups);
  if (dtype == SVF_F32) {
    if (p.d == 64) hipLaunchKernelGGL((verify_attn_valu_kernel<float, 64>), grid, dim3(kThreads), 0, st, p, row_groups);
    else hipLaunchKernelGGL((verify_attn_valu_kernel<float, 128>), grid, dim3(kThreads), 0, st, p, row_groups);
  } else {
    if (p.d == 64) hipLaunchKernelGGL((verify_attn_valu_kernel<__hip_bfloat16, 64>), grid, dim3(kThreads), 0, st, p, row_groups);
    else hipLaunchKernelGGL((verify_attn_valu_kernel<__hip_bfloat16, 128>), grid, dim3(kThreads), 0, st, p, row_groups);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_merge_splits(p, dtype, st);
}

}  // namespace svf
